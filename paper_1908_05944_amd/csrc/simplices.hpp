// Candidate triangles and tetrahedra and the pruning (Steps 1-5), for gfx950.
//
// Every simplex belongs to its vertex with the least input id, so the work is
// laid out by ball: a block takes a group of consecutive balls (in sorted
// order), whose candidate edges are consecutive (upper rows, ordered by input
// id), and enumerates and tests all simplices of those balls. With the rows in
// id order, each ball's simplices come out in output order, so the emit needs
// no sort.
//
// A candidate triangle of ball i is a pair (j, k) of its upper row whose own
// grown spheres cross (tested from the two balls, no search in j's row) and
// which passes AC3; a candidate tetrahedron is a pair (i, j, k), (i, j, l) of
// candidate triangles of one edge with k and l crossing. Both are pair
// problems over short rows: the pairs of a block are spread evenly over its
// threads (a thread per row entry, looping over the entries after it, would
// hold up its wave for the longest row), the survivors of each test are
// compacted in LDS before the next test, so that the float64 tests run in full
// waves, and the order of the pairs is kept throughout.
//
// Triangles of group g are stored densely from pair_base[g] on, which leaves
// room for every pair (about 3.8 per candidate triangle at 0.05 atoms per A^3
// and alpha = 0): no count, scan or compaction pass, and no read-back of the
// triangle total. Where the pairs are too many the host counts the triangles
// first and passes their scan instead. Tetrahedra of a group go to a slab of
// fixed size, or to counted ranges if a group outgrew its slab.
//
// The AC2 tests (walks along neighbour rows, a thread per simplex) are kernels
// of their own: beside the pair machinery they would hold far more registers
// (194 against 64), and a block's few tetrahedra would wait on its triangles.
#pragma once
#include "kernels.hpp"

namespace acx {

constexpr int PAIR_WIN = 2048;  // pairs of a block worked on at a time
constexpr int NWAVE = BLOCK / WAVE;

// Candidate arrays of one build. Edge e: owner edge_i[e], other end up[e]
// (sorted indices) with input id up_id[e]. Triangle t: edges tri_e[t] = (i, j)
// and tri_f[t] = (i, k), so k = up[tri_f[t]]. A group is 2^gshift consecutive
// balls (at most GROUP); group g's triangles are [tri_base[g], tri_base[g] +
// tri_cnt[g]).
struct Cands {
    const int4 *atom;
    const int *perm;
    const int *nbr_start, *nbr_cnt, *nbr;
    const int *up_start, *up, *up_id, *edge_i;
    const int *tri_base;
    int *tri_cnt, *tri_e, *tri_f;
    int *tri_first;  // first triangle of an edge, where it has any
    int *tri_sub;    // first triangle of each 2^sshift balls (sshift <= gshift)
    int n, gshift, sshift;
};

// The pairs (a, b), a < b, of entries of one row, for the PT consecutive
// entries a of each thread of the block: entry u has later[u] later entries
// in its row. Pairs are numbered entry by entry; `own` and `soff` (LDS) map a
// pair of the window [w0, w0 + PAIR_WIN) back to its entry. Ends with a barrier.
template <int PT>
__device__ __forceinline__ void pair_owners(int w0, int off, const int (&later)[PT], unsigned short *own) {
#pragma unroll
    for (int u = 0; u < PT; u++) {
        const int lo = max(off, w0), hi = min(off + later[u], w0 + PAIR_WIN);
#pragma unroll 1
        for (int p = lo; p < hi; p++) own[p - w0] = (unsigned short)(threadIdx.x * PT + u);
        off += later[u];
    }
    __syncthreads();
}
// Exclusive scan of the entries' pair counts, into soff (no barrier after);
// returns the thread's first and sets the block's total.
template <int PT>
__device__ __forceinline__ int pair_scan(const int (&later)[PT], int *soff, int *total) {
    int s = 0;
#pragma unroll
    for (int u = 0; u < PT; u++) s += later[u];
    const int off = block_exclusive_scan<BLOCK>(s, total);
    int run = off;
#pragma unroll
    for (int u = 0; u < PT; u++) {
        soff[threadIdx.x * PT + u] = run;
        run += later[u];
    }
    return off;
}

// Index of the wave in its block, known to be the same in all its lanes.
__device__ __forceinline__ int wave_id() { return __builtin_amdgcn_readfirstlane((int)threadIdx.x / WAVE); }

// Ordered compaction across a block: the waves take contiguous parts of
// [0, m) of `part` items each (a multiple of WAVE), f(x, v) tests item x (v:
// what is stored for it), and the items it accepts are stored, in order, at
// out[part * wave ...]. Returns the wave's number of accepted items.
template <class F>
__device__ __forceinline__ int wave_filter(int m, int part, unsigned short *out, F &&f) {
    const int lane = lane_id(), w = wave_id();
    const int s0 = min(w * part, m), s1 = min(s0 + part, m);
    int h = 0;
#pragma unroll 1
    for (int x0 = s0; x0 < s1; x0 += WAVE) {
        const int x = x0 + lane;
        int v = 0;
        const bool pass = x < s1 && f(x, v);
        const unsigned long long mask = __ballot(pass);
        if (pass) out[w * part + h + __popcll(mask & ((1ull << lane) - 1ull))] = (unsigned short)v;
        h += __popcll(mask);
    }
    return h;
}
__device__ __forceinline__ int part_of(int m) { return ((m + NWAVE - 1) / NWAVE + WAVE - 1) / WAVE * WAVE; }

// The items that wave_filter left in NWAVE parts, seen as one list.
struct Parts {
    int before[NWAVE], total, part;
    __device__ __forceinline__ void load(const int *wtot, int part_) {
        part = part_;
        total = 0;
#pragma unroll
        for (int w = 0; w < NWAVE; w++) {
            before[w] = total;
            total += __builtin_amdgcn_readfirstlane(wtot[w]);
        }
    }
    __device__ __forceinline__ int slot(int x) const {
        int w = 0;
#pragma unroll
        for (int k = 1; k < NWAVE; k++) w += x >= before[k];
        int b = 0;
#pragma unroll
        for (int k = 0; k < NWAVE; k++) b = w == k ? before[k] : b;
        return w * part + (x - b);
    }
};

// Edge of ball a to the ball of input id `id` in a's upper row; -1 if absent.
__device__ __forceinline__ int find_edge(const Cands &cd, int a, int id) {
    int lo = cd.up_start[a], hi = cd.up_start[a + 1] - 1;
    while (lo <= hi) {
        const int mid = (lo + hi) >> 1;
        const int v = cd.up_id[mid];
        if (v == id) return mid;
        if (v < id) lo = mid + 1; else hi = mid - 1;
    }
    return -1;
}

// Triangle with edges (e, f) of group g; -1 if absent. tri_first[e] is the
// first triangle of edge e, where it has any; a row of triangles ascends by f.
__device__ __forceinline__ int find_tri(const Cands &cd, int g, int e, int f) {
    const int t0 = cd.tri_base[g], t1 = t0 + cd.tri_cnt[g];
    int t = cd.tri_first[e];
    if (t < t0) return -1;
#pragma unroll 1
    while (t < t1 && cd.tri_e[t] == e && cd.tri_f[t] < f) t++;
    return t < t1 && cd.tri_e[t] == e && cd.tri_f[t] == f ? t : -1;
}

// Edges of ball a to the balls of input ids `id1` < `id2`, -1 where absent:
// a walk along a's upper row, four entries at a time.
__device__ __forceinline__ int2 find_edges(const Cands &cd, int a, int id1, int id2) {
    const int e0 = cd.up_start[a], e1 = cd.up_start[a + 1];
    int2 r = make_int2(-1, -1);
    for (int e = e0; e < e1 && r.y < 0; e += 4) {
        int v[4];
#pragma unroll
        for (int u = 0; u < 4; u++) v[u] = cd.up_id[min(e + u, e1 - 1)];
#pragma unroll
        for (int u = 0; u < 4; u++) {
            if (v[u] == id1) r.x = min(e + u, e1 - 1);
            if (v[u] == id2) r.y = min(e + u, e1 - 1);
        }
        if (v[3] > id2) break;
    }
    return r;
}

constexpr int AC2_GROUP = 4;  // neighbours loaded together in the AC2 loops
// Neighbour arrays are allocated AC2_GROUP entries longer, so that a group
// that starts inside a row (or at its end) can be loaded whole (entries past
// the row are replaced, not used).
constexpr int NBR_PAD = AC2_GROUP;

// The AC2 tests below walk ball i's neighbour row in float32 (power_of), in
// groups of AC2_GROUP neighbours whose loads are issued together. `own` of the
// row's balls are the simplex's, undecided by themselves, as are the entries
// that fill up the last group (i itself: b = 0, gamma = 0, P = 0), so the
// undecided ones are counted and none is compared with the simplex's balls.
// Where no violator is certain but more are undecided (near ties: 18 of 2.2
// million triangles of 20,000 atoms with solvent-accessible radii), the row is
// walked once more with the float64 filter and the exact test.
// f(r, P, k): called with each neighbour's {b, gamma}, its power and its place
// in the row. STOP: end after the first group with a violator.
// Two forms: the row as {b, gamma} about i in LDS (RowLds, of many simplices of
// one ball), or gathered from memory.
enum { AC2_HOLDS = 0, AC2_VIOLATED = 1, AC2_UNSURE = 2 };
// status of a face; AC2 leaves 0 or 1
enum { FACE_OUT = 0, FACE_GABRIEL = 1, FACE_ATTACHED = 2, FACE_UNSURE = 3 };
struct RowLds {
    const float4 *row;  // filled up with zeros to a multiple of AC2_GROUP
    int len;
    __device__ __forceinline__ unsigned places() const { return 255u; }  // mask of a place in the row
    __device__ __forceinline__ void begin() {}
    __device__ __forceinline__ void load(int k, float4 (&r)[AC2_GROUP]) {
#pragma unroll
        for (int u = 0; u < AC2_GROUP; u++) r[u] = row[k + u];
    }
};
struct RowMem {
    const int4 *atom;
    const int *row;
    int i, len;
    int4 me;
    int nx[AC2_GROUP];  // the next group's indices, one 16-byte load while this group is tested
    __device__ __forceinline__ RowMem(const Cands &cd, int i_)
        : atom(cd.atom), row(cd.nbr + cd.nbr_start[i_]), i(i_), len(cd.nbr_cnt[i_]) {}
    __device__ __forceinline__ unsigned places() const { return len <= 256 ? 255u : 8191u; }
    __device__ __forceinline__ void begin() {
        me = atom[i];
        __builtin_memcpy(nx, row, sizeof nx);  // in bounds: NBR_PAD
    }
    __device__ __forceinline__ void load(int k, float4 (&r)[AC2_GROUP]) {
        int4 q[AC2_GROUP];
#pragma unroll
        for (int u = 0; u < AC2_GROUP; u++) q[u] = atom[k + u < len ? nx[u] : i];
        __builtin_memcpy(nx, row + (k + AC2_GROUP < len ? k + AC2_GROUP : k), sizeof nx);  // the last group reloads itself
#pragma unroll
        for (int u = 0; u < AC2_GROUP; u++) r[u] = relative_ball(me, q[u]);
    }
};
template <bool STOP, class R, class F>
__device__ __forceinline__ int walk_row(R row, const Power32 &pw, int own, F &&f) {
    bool viol = false;
    int undecided = 0;
    row.begin();
    for (int k = 0; k < row.len; k += AC2_GROUP) {
        float4 r[AC2_GROUP];
        row.load(k, r);
#pragma unroll
        for (int u = 0; u < AC2_GROUP; u++) {
            const float P = power_of(pw, r[u]);
            viol |= P < -pw.e;
            undecided += fabsf(P) <= pw.e;
            f(r[u], P, k + u);
        }
        if (STOP && viol) break;
    }
    if (viol) return AC2_VIOLATED;
    return undecided == own + (-row.len & (AC2_GROUP - 1)) ? AC2_HOLDS : AC2_UNSURE;
}

// AC2 of candidate edge (i, j) at its own ortho-centre (Step 4): every violator
// meets the ortho-centre, so it is in i's neighbour row. Every neighbour is
// tested (no early exit: most edges pass, and the loop stays convergent).
template <class R>
__device__ __forceinline__ int edge_ac2(const PredParams &pp, R row, const int4 &vi, const int4 &vj) {
    if (pp.force_exact) return AC2_UNSURE;
    // P = |a|^2 gamma - beta (a.b)
    const Edge ed = edge_setup(vi, vj);
    const float den = (float)ed.den, be = (float)ed.beta;
    Power32 pw{den, be * (float)ed.ax, be * (float)ed.ay, be * (float)ed.az, 0.0f};
    pw.e = 16.0f / (1 << 24) * fmaf(den, (float)pp.gmax, (float)pp.bmax * (fabsf(pw.mx) + fabsf(pw.my) + fabsf(pw.mz)));
    return walk_row<false>(row, pw, 1, [](const float4 &, float, int) {});
}
__device__ __forceinline__ bool edge_violated(const Cands &cd, const PredParams &pp, int i, int j) {
    const Edge ed = edge_setup(cd.atom[i], cd.atom[j]);
    const int ns = cd.nbr_start[i], ne = ns + cd.nbr_cnt[i];
    bool viol = false;
#pragma unroll 1
    for (int p = ns; p < ne && !viol; p++) {
        const int q = cd.nbr[p];
        viol = q != j && edge_violation_sign(ed, i, j, cd.atom[q], q, cd.perm, pp.force_exact) < 0;
    }
    return viol;
}

// The rows of simplices that float32 left undecided: whether a ball of row [p, ne)
// that is not the simplex's own violates it. filter(ball) gives the float64 sign, 0
// where exact(ball, its place in the order) has to decide. Each lane goes on to its
// next undecided ball before any decides one: the lanes of a wave have theirs at
// different places of their rows, and the exact test in the loop over the row ran
// for a lane or two at a time (builds of lattices with ties everywhere: 104,000 balls
// 664 us, 4,515 so; 51,000 with 10 million ties 5,150, 28,500 so).
template <class OWN, class FILTER, class EXACT>
__device__ __forceinline__ bool row_violated(const Cands &cd, int p, int ne, OWN &&own, FILTER &&filter, EXACT &&exact) {
#pragma unroll 1
    for (;;) {
        int q = 0, sg = 1;
        int4 aq = make_int4(0, 0, 0, 0);
#pragma unroll 1
        while (p < ne && sg > 0) {
            q = cd.nbr[p++];
            if (own(q)) continue;
            aq = cd.atom[q];
            sg = filter(aq);
        }
        if (sg == 0) sg = exact(aq, q);
        else if (sg > 0) return false;  // the row's end
        if (sg < 0) return true;
    }
}

// OrthoSize evaluated with the vertices in lexicographic order of their
// integer centres (a total order: equal centres are rejected). The rounded
// float64 value then depends only on the balls, not on the grid, the sorted
// order or the other molecules of a batch, so reported Sizes are
// bit-identical whatever the cell size; no input-index gather is needed.
__device__ __forceinline__ bool centre_less(const int4 &a, const int4 &b) {
    return a.x != b.x ? a.x < b.x : (a.y != b.y ? a.y < b.y : a.z < b.z);
}

__device__ __forceinline__ double edge_size_canon(int4 a, int4 b) {
    return centre_less(a, b) ? edge_orthosize(edge_setup(a, b)) : edge_orthosize(edge_setup(b, a));
}

template <int K>
__device__ __forceinline__ void sort_centres(int4 (&v)[K]) {
#pragma unroll
    for (int a = 1; a < K; a++)
#pragma unroll
        for (int b = a; b > 0; b--)
            if (centre_less(v[b], v[b - 1])) {
                const int4 u = v[b]; v[b] = v[b - 1]; v[b - 1] = u;
            }
}

__device__ __forceinline__ double tet_size_canon(int4 a, int4 b, int4 c, int4 d, const PredParams &pp) {
    int4 v[4] = {a, b, c, d};
    sort_centres<4>(v);
    return tet_orthosize(tet_setup(v[0], v[1], v[2], v[3], pp));
}

// AC2 of candidate triangle t = (i, j, k) at its own ortho-centre (Step 3;
// violators are in i's neighbour row) and its OrthoSize (tsize[t]). Every
// neighbour is tested (no early exit, convergent loop). The triangle is set up
// once, in the order of its Size; relative to ball i, whose distances to its
// neighbours are bounded, M is that of the order's first ball moved by
// 2 |n|^2 (v0 - v_i).
// APEX: also two neighbours that rule out most tetrahedra on the triangle. The
// ortho-centres of all balls with the triangle lie on its axis, c_t + s n up to
// a scale; ball q, at signed distance D = n.b from the plane, violates a centre
// iff P_q - s D < 0, so on its side of the plane the ball of least P / D (where
// D > 0; of the largest where D < 0) violates every tetrahedron of another
// apex there. The two are found in float32, their places in the row in the low
// 8 bits of the quotient, 13 of rows past 256 neighbours (past 8,192 another one of
// the row; with 8 bits for all, 2,598 grown balls around one took 38 ms, 20 in the
// walks of the candidates that were left): they are only the first neighbours that
// a candidate is tested against, with the exact predicate.
template <bool APEX, class R>
__device__ __forceinline__ int tri_ac2(const PredParams &pp, R row, const int4 &vi, const int4 &vj, const int4 &vk,
                                       double &size, int2 &apex) {
    int4 v[3] = {vi, vj, vk};
    sort_centres<3>(v);
    const Tri ts = tri_setup(v[0], v[1], v[2], pp);
    size = tri_orthosize(ts);
    apex = make_int2(-1, -1);
    if (pp.force_exact) return AC2_UNSURE;
    const double den = (double)ts.den, den2 = 2.0 * den;
    const double Mx = ts.Mx + den2 * (double)(v[0].x - vi.x), My = ts.My + den2 * (double)(v[0].y - vi.y),
                 Mz = ts.Mz + den2 * (double)(v[0].z - vi.z);
    const Power32 pw = power32(den, Mx, My, Mz, ts.eP, pp);
    const float nx = (float)ts.nx, ny = (float)ts.ny, nz = (float)ts.nz;
    float lo = INFINITY, hi = -INFINITY;
    const unsigned place = row.places();
    const int res = walk_row<false>(row, pw, 2, [&](const float4 &r, float P, int at) {
        if (APEX) {
            const float D = fmaf(nx, r.x, fmaf(ny, r.y, nz * r.z));
            const float s = __uint_as_float((__float_as_uint(P * __builtin_amdgcn_rcpf(D)) & ~place) | (at & place));
            const bool other = fabsf(P) > pw.e;
            lo = fminf(lo, other & (D > 0.0f) ? s : INFINITY);
            hi = fmaxf(hi, other & (D < 0.0f) ? s : -INFINITY);
        }
    });
    if (lo < INFINITY) apex.x = __float_as_uint(lo) & place;
    if (hi > -INFINITY) apex.y = __float_as_uint(hi) & place;
    return res;
}
__device__ __forceinline__ bool tri_violated(const Cands &cd, const PredParams &pp, int i, int j, int k, Counters *cnt) {
    const Tri tr = tri_setup(cd.atom[i], cd.atom[j], cd.atom[k], pp);
    const int ns = cd.nbr_start[i];
    return row_violated(
        cd, ns, ns + cd.nbr_cnt[i], [&](int q) { return q == j || q == k; },
        [&](const int4 &aq) { return pp.force_exact ? 0 : tri_violation_filter(tri_filter(tr), aq); },
        [&](const int4 &aq, int q) {
            if (!pp.force_exact) note_fallback(cnt);
            return tri_violation_exact(tr, i, j, k, aq, q, cd.perm);
        });
}

// AC2 of tetrahedron (i, j, k, l) against i's neighbour row, ending at the
// first violator (most candidates of large radii fail within a few).
__device__ __forceinline__ bool tet_ac2(const Cands &cd, const Tet &ts, const PredParams &pp, int i, int j, int k,
                                        int l, Counters *cnt) {
    int res = AC2_UNSURE;
    if (!pp.force_exact) {
        // P = sign(D) (D gamma - M.b)
        const double sD = ts.D > 0 ? 1.0 : -1.0;
        const Power32 pw = power32(fabs((double)ts.D), sD * ts.Mx, sD * ts.My, sD * ts.Mz, ts.eP, pp);
        res = walk_row<true>(RowMem(cd, i), pw, 3, [](const float4 &, float, int) {});
    }
    bool viol = res == AC2_VIOLATED;
    if (res == AC2_UNSURE) {
        const int io = opaque(i);
        const Tet te = tet_setup(cd.atom[io], cd.atom[j], cd.atom[k], cd.atom[l], pp);
        const int ns = cd.nbr_start[io];
        viol = row_violated(
            cd, ns, ns + cd.nbr_cnt[io], [&](int q) { return q == j || q == k || q == l; },
            [&](const int4 &aq) { return pp.force_exact ? 0 : tet_violation_filter(tet_filter(te), aq); },
            [&](const int4 &aq, int q) {
                if (!pp.force_exact) note_fallback(cnt);
                return tet_violation_exact(te, i, j, k, l, aq, q, cd.perm);
            });
    }
    return !viol;
}

// ---------------------------------------------------------------------------
// Candidate triangles (Sec. 4.3) of a group's edges. The balls of EDGE_CH
// edges' other ends (and of the next EDGE_AHEAD, where a row goes on) are held
// in LDS, so that the pair tests wait for no memory. COUNT: the groups' totals
// only (the first pass of a counted build). Bound by instruction issue (half of
// the time) and the barriers between the tests: 195 us at 3M atoms and alpha = 0
// with 512 edges at a time; with 256 208, with 1,024 240.
// LONG (rows longer than the slots, after a counted neighbour search): the third
// balls of (i, j) are also among the upper entries of j. Where more than LONG_ROW
// edges come after (i, j) in its row and j has fewer, j's are the items, each
// looked up in i's row: a large ball with thousands of small ones around it has a
// few items an edge instead of thousands (7.9 A among 2,942 of 0.45 A: 65 ms with
// all pairs, 0.33 as this). Looked for where the edges held have LONG_PAIRS pairs.
// (In every build, the test of has_long costs 0.8 % at 3M atoms.)
constexpr int EDGE_PT = 2, EDGE_CH = EDGE_PT * BLOCK, EDGE_AHEAD = 64;
constexpr int LONG_ROW = 64, LONG_PAIRS = 4 * PAIR_WIN;
static_assert(EDGE_CH == EDGES_HELD && LONG_PAIRS == PAIRS_LONG, "later_counted");
constexpr int LONG_EDGE = 0x80;  // in part_no: the items of the edge are j's upper entries
template <bool COUNT, bool LONG>
__global__ void __launch_bounds__(BLOCK) k_triangles(Cands cd, PredParams pp, long long *__restrict__ tri_min, Counters *cnt,
                                                      const int *__restrict__ stop) {
    if (stop && *stop) return;
    __shared__ int4 sat[EDGE_CH + EDGE_AHEAD];
    __shared__ unsigned short own[PAIR_WIN], hit[PAIR_WIN], res[PAIR_WIN];
    __shared__ int soff[EDGE_CH];
    __shared__ unsigned char part_no[EDGE_CH];  // part of the group an edge belongs to (at most 64), LONG_EDGE
    __shared__ int wtot[2][NWAVE];
    const int g = xcd_block();
    const int b0 = g << cd.gshift, b1 = min(b0 + (1 << cd.gshift), cd.n);
    const int e0 = cd.up_start[b0], e1 = cd.up_start[b1];
    const int w = wave_id(), lane = lane_id();
    int out = COUNT ? 0 : cd.tri_base[g];
    const int out0 = out;
    int last_part = -1;  // part of the last triangle so far
    int *const sub = COUNT ? nullptr : cd.tri_sub + (b0 >> cd.sshift);
    for (int c0 = e0; c0 < e1; c0 += EDGE_CH) {
        for (int x = threadIdx.x; x < min(EDGE_CH + EDGE_AHEAD, e1 - c0); x += BLOCK) sat[x] = cd.atom[cd.up[c0 + x]];
        int later[EDGE_PT];
#pragma unroll
        for (int u = 0; u < EDGE_PT; u++) {
            const int e = c0 + threadIdx.x * EDGE_PT + u;
            const int i = e < e1 ? cd.edge_i[e] : 0;
            later[u] = e < e1 ? cd.up_start[i + 1] - e - 1 : 0;
            part_no[threadIdx.x * EDGE_PT + u] = (unsigned char)((i - b0) >> cd.sshift);
        }
        int pairs, some[EDGE_PT];
#pragma unroll
        for (int u = 0; u < EDGE_PT; u++) some[u] = LONG ? later_counted(later[u]) : later[u];
        int off = pair_scan<EDGE_PT>(some, soff, &pairs);
        const bool has_long = LONG && pairs > LONG_PAIRS;
        if (has_long) {
#pragma unroll
            for (int u = 0; u < EDGE_PT; u++) {
                if (later[u] <= LONG_ROW) continue;
                const int x = threadIdx.x * EDGE_PT + u, j = cd.up[c0 + x];
                const int items = cd.up_start[j + 1] - cd.up_start[j];
                if (items >= later[u]) continue;
                later[u] = items;
                part_no[x] |= LONG_EDGE;
            }
            off = pair_scan<EDGE_PT>(later, soff, &pairs);
        }
        int prev = -1;  // edge (less c0) of the last triangle of the windows before
        // edge (less c0) of i to the k-th upper entry of j, for edge c0 + o = (i, j); -1 if there is none
        auto joint = [&](int o, int k) {
            const int e = c0 + o, id = cd.up_id[cd.up_start[cd.up[e]] + k];
            int lo = e + 1, hi = cd.up_start[cd.edge_i[e] + 1];
            const int end = hi;
            while (lo < hi) {
                const int mid = (lo + hi) >> 1;
                if (cd.up_id[mid] < id) lo = mid + 1; else hi = mid;
            }
            return lo < end && cd.up_id[lo] == id ? lo - c0 : -1;
        };
        auto part_of_edge = [&](int x) { return LONG ? part_no[x] & ~LONG_EDGE : part_no[x]; };
        // the ball at the far end of edge c0 + x
        auto far_ball = [&](int x) { return x < EDGE_CH + EDGE_AHEAD ? sat[x] : cd.atom[cd.up[c0 + x]]; };
        for (int w0 = 0; w0 < pairs; w0 += PAIR_WIN) {
            pair_owners<EDGE_PT>(w0, off, later, own);
            const int wn = min(PAIR_WIN, pairs - w0);
            // second edge of pair x of the window, less c0 (the first is own[x])
            auto second = [&](int x) {
                const int o = own[x], k = w0 + x - soff[o];
                return has_long && (part_no[o] & LONG_EDGE) ? joint(o, k) : o + 1 + k;
            };
            // pairs of the upper row whose spheres cross
            const int p1 = part_of(wn);
            const int h = wave_filter(wn, p1, hit, [&](int x, int &v) {
                v = x;
                const int y = second(x);
                if (has_long && y < 0) return false;
                return spheres_cross(far_ball(own[x]), far_ball(y), pp);
            });
            if (lane == 0) wtot[0][w] = h;
            __syncthreads();
            // AC3 of those
            Parts hs;
            hs.load(wtot[0], p1);
            const int p2 = part_of(hs.total);
            const int r = wave_filter(hs.total, p2, res, [&](int x, int &v) {
                v = hit[hs.slot(x)];
                const int o = own[v];
                return tri_candidate(cd.atom[cd.edge_i[c0 + o]], far_ball(o), far_ball(second(v)), pp, cnt);
            });
            if (lane == 0) wtot[1][w] = r;
            __syncthreads();
            Parts rs;
            rs.load(wtot[1], p2);
            if (!COUNT) {
                for (int x = threadIdx.x; x < rs.total; x += BLOCK) {
                    const int v = res[rs.slot(x)];
                    const int o = own[v];
                    cd.tri_e[out + x] = c0 + o;
                    cd.tri_f[out + x] = c0 + second(v);
                    tri_min[out + x] = ORDERED_POS_INF;  // no kept coface yet
                    // the edge's first triangle (an edge cut by the window sets it
                    // in the window of its first), and that of each part from the
                    // one after its predecessor's on
                    const int before = x > 0 ? own[res[rs.slot(x - 1)]] : prev;
                    if (before != o) {
                        cd.tri_first[c0 + o] = out + x;
                        for (int k = x > 0 ? part_of_edge(before) + 1 : last_part + 1; k <= part_of_edge(o); k++)
                            sub[k] = out + x;
                    }
                }
            }
            if (rs.total > 0) {
                prev = own[res[rs.slot(rs.total - 1)]];
                last_part = part_of_edge(prev);
            }
            out += rs.total;
            __syncthreads();
        }
        __syncthreads();  // sat and soff are rewritten by the next round
    }
    if (threadIdx.x == 0) cd.tri_cnt[g] = out - out0;
    if (!COUNT)
        for (int k = last_part + 1 + threadIdx.x; k << cd.sshift < b1 - b0; k += BLOCK) sub[k] = out;
}

// ---------------------------------------------------------------------------
// A face that passes AC2 itself is in K with Size = OrthoSize whatever its
// cofaces do, so only faces failing AC2 record the kept coface: the least
// Size of their kept cofaces (order-preserving integer; +inf while none), so
// such a face is kept iff that minimum is finite.
// gab: the faces' status.
__device__ __forceinline__ void mark_face(const unsigned char *gab, long long *mins, int f, long long key,
                                          Counters *cnt) {
    if (f < 0) { atomicOr(&cnt->lookup, 1); return; }
    if (gab[f] == FACE_GABRIEL) return;
    atomicMin(&mins[f], key);
}

// The four facets of tetrahedron (t, t2), t = (i, j, k), t2 = (i, j, l): t,
// t2, (i, k, l) (of the same group g) and (j, k, l) (of ball j's group).
__device__ __forceinline__ int4 tet_facets(const Cands &cd, int g, int t, int t2) {
    const int e = cd.tri_e[t], f = cd.tri_f[t], f2 = cd.tri_f[t2];
    const int j = cd.up[e];
    const int a = find_tri(cd, g, f, f2);
    const int2 r = find_edges(cd, j, cd.up_id[f], cd.up_id[f2]);
    const int b = r.x < 0 || r.y < 0 ? -1 : find_tri(cd, j >> cd.gshift, r.x, r.y);
    return make_int4(t, t2, a, b);
}

// AC2 of the candidate edges and triangles, and the triangles' OrthoSize. A
// block takes a part of a group, 2^sshift consecutive balls (at most AC2_ROWS /
// SLOT), and puts their neighbour rows in LDS as {b, gamma}: 7 neighbours a ball
// are gathered and made relative once instead of once per simplex (3.5 edges
// and 2 triangles a ball at alpha = 0, 21 and 110 with solvent-accessible
// radii: gathers of a line each were what bound the edges' test), and a test
// costs 8 instructions a neighbour against 27 in integers and float64. Rows
// start SLOT + 1 entries apart (other banks; the last entry holds the length).
// Waves take 64 triangles or 64 edges each. Bound by instruction issue (two
// thirds; the triangles' float64 setup most of it) and by the chain of loads
// before the walk, so the first simplex of each thread is loaded along with the
// rows, level by level. Eight waves per SIMD: the walk needs less than 64
// registers; a simplex that it leaves undecided is marked and looked at again
// at the end (inside the loop, the exact test's registers were spilled around
// it by every wave: 390 us).
// Both tests at 3M atoms and alpha = 0: 308 us as two kernels without LDS, 222
// as this; 100,000 atoms with solvent-accessible radii 1,150 and 412. With rows
// gathered from a float4 copy of the balls (16 bytes a ball more to write and
// hold) 239 and 417, and of that 512 threads 285 and 405, 512 entries 261 and 416,
// with 128 threads 250 and 442.
// SLOT = 0: rows of any length (after a counted neighbour search), gathered per
// simplex. Without rows of its own a part need not be one block's: gridDim.y
// blocks share it (rows_split), so that a ball with thousands of simplices does
// not leave the rest of the GPU idle (a build of a ball of 7.9 A among 2,942 of
// 0.45 A 17 ms shorter; 300 balls of 6.2 A 4.6 ms against 5.8). `what`: bit 0
// edges, bit 1 triangles.
constexpr int AC2_BLOCK = 256;
constexpr int AC2_ROWS = 1024;
enum { AC2_EDGES = 1, AC2_TRIANGLES = 2 };
// What the tests write: status of edges and triangles, least Size of a kept
// coface of an edge that fails, balls that own one, Size and apex balls of the
// triangles.
struct Ac2Out {
    unsigned char *egab;
    long long *edge_min;
    unsigned char *eng;
    unsigned char *tgab;
    double *tsize;
    int2 *apex;
};
template <int SLOT>
constexpr int ac2_rows() { return SLOT ? AC2_ROWS / (SLOT ? SLOT : 1) * (SLOT + 1) : 1; }
template <int SLOT, bool APEX>
__device__ __forceinline__ void ac2_part(const Cands &cd, const PredParams &pp, int part, int what, const Ac2Out &o,
                                         Counters *cnt, float4 *rows) {
    constexpr int STRIDE = SLOT + 1, PT = AC2_ROWS / AC2_BLOCK;
    const int b0 = part << cd.sshift, b1 = min(b0 + (1 << cd.sshift), cd.n);
    const int g = b0 >> cd.gshift;
    const int lane = lane_id();
    // the block's edges and triangles, and its rows
    const int e0 = cd.up_start[b0], e1 = cd.up_start[b1];
    const int t0 = cd.tri_sub[part];
    const int t1 = b1 < cd.n && b1 >> cd.gshift == g ? cd.tri_sub[part + 1] : cd.tri_base[g] + cd.tri_cnt[g];
    int len[PT], ns[PT];
    if (SLOT) {
#pragma unroll
        for (int r = 0; r < PT; r++) {
            const int b = min(b0 + ((int)threadIdx.x + r * AC2_BLOCK) / (SLOT ? SLOT : 1), b1 - 1);
            len[r] = min(cd.nbr_cnt[b], SLOT);
            ns[r] = cd.nbr_start[b];
        }
    }
    const int tw = what & AC2_TRIANGLES ? (t1 - t0 + WAVE - 1) / WAVE : 0;
    const int ew = what & AC2_EDGES ? (e1 - e0 + WAVE - 1) / WAVE : 0;
    // a thread's simplex of wave item w (x < 0: none): first a triangle's edges
    // or an edge's ends, then a triangle's ends, then the balls
    struct Item {
        int x, i, j, k;
        int4 vi, vj, vk;
    };
    auto fetch_ids = [&](int w) {
        Item it;
        it.x = -1;
        if (w < tw) {
            const int x = t0 + w * WAVE + lane;
            if (x < t1) {
                it.x = x;
                it.i = cd.tri_e[x];
                it.k = cd.tri_f[x];
            }
        } else if (w < tw + ew) {
            const int x = e0 + (w - tw) * WAVE + lane;
            if (x < e1) {
                it.x = x;
                it.i = cd.edge_i[x];
                it.j = cd.up[x];
            }
        }
        return it;
    };
    auto fetch_ends = [&](int w, Item &it) {
        if (w < tw && it.x >= 0) {
            const int e = it.i;
            it.i = cd.edge_i[e];
            it.j = cd.up[e];
            it.k = cd.up[it.k];
        }
    };
    auto fetch_balls = [&](int w, Item &it) {
        if (it.x < 0) return;
        it.vi = cd.atom[it.i];
        it.vj = cd.atom[it.j];
        if (w < tw) it.vk = cd.atom[it.k];
    };
    // the block's waves among those of the part
    const int w0 = SLOT ? wave_id() : (int)blockIdx.y * (AC2_BLOCK / WAVE) + wave_id();
    const int waves = SLOT ? AC2_BLOCK / WAVE : (int)gridDim.y * (AC2_BLOCK / WAVE);
    int w = w0;
    Item it = fetch_ids(w);
    if constexpr (SLOT != 0) {
        int q[PT];
#pragma unroll
        for (int r = 0; r < PT; r++) {
            const int k = ((int)threadIdx.x + r * AC2_BLOCK) % SLOT;
            q[r] = k < len[r] ? cd.nbr[ns[r] + k] : -1;
        }
        fetch_ends(w, it);
#pragma unroll
        for (int r = 0; r < PT; r++) {
            const int y = (int)threadIdx.x + r * AC2_BLOCK, b = y / SLOT, k = y % SLOT;
            if (b0 + b < b1 && k < len[r] + (-len[r] & (AC2_GROUP - 1)))
                rows[b * STRIDE + k] = relative_ball(cd.atom[b0 + b], cd.atom[q[r] < 0 ? b0 + b : q[r]]);
            if (k == 0) rows[b * STRIDE + SLOT].x = __int_as_float(len[r]);
        }
        fetch_balls(w, it);
        __syncthreads();
    } else {
        fetch_ends(w, it);
        fetch_balls(w, it);
    }
    auto row_of = [&](int i) {
        if constexpr (SLOT != 0) return RowLds{rows + (i - b0) * STRIDE, __float_as_int(rows[(i - b0) * STRIDE + SLOT].x)};
        else return RowMem(cd, i);
    };
    // an edge's verdict; one that fails starts o.edge_min[e] (the least Size of a
    // kept coface) and flags its owner in eng
    auto edge_is = [&](int e, int i, bool viol) {
        o.egab[e] = (unsigned char)!viol;
        if (viol) {
            o.edge_min[e] = ORDERED_POS_INF;
            o.eng[i] = 1;
        }
    };
    bool unsure = false;
#pragma unroll 1
    while (w < tw + ew) {
        const int x = it.x;
        if (x >= 0) {
            if (w < tw) {
                double size;
                int2 at;
                const int res = tri_ac2<APEX>(pp, row_of(it.i), it.vi, it.vj, it.vk, size, at);
                o.tsize[x] = size;
                o.tgab[x] = res == AC2_UNSURE ? FACE_UNSURE : (unsigned char)(res == AC2_HOLDS);
                unsure |= res == AC2_UNSURE;
                if (APEX) {  // j: none
                    const int *nb = cd.nbr + cd.nbr_start[it.i];
                    o.apex[x] = make_int2(at.x < 0 ? it.j : nb[at.x], at.y < 0 ? it.j : nb[at.y]);
                }
            } else {
                const int res = edge_ac2(pp, row_of(it.i), it.vi, it.vj);
                if (res == AC2_UNSURE) o.egab[x] = FACE_UNSURE;
                else edge_is(x, it.i, res == AC2_VIOLATED);
                unsure |= res == AC2_UNSURE;
            }
        }
        w += waves;
        it = fetch_ids(w);
        fetch_ends(w, it);
        fetch_balls(w, it);
    }
    // each wave's own undecided ones, once more
    if (!__any(unsure)) return;
#pragma unroll 1
    for (w = w0; w < tw + ew; w += waves) {
        Item un = fetch_ids(w);
        fetch_ends(w, un);
        if (un.x < 0) continue;
        if (w < tw) {
            if (o.tgab[un.x] == FACE_UNSURE) o.tgab[un.x] = (unsigned char)!tri_violated(cd, pp, un.i, un.j, un.k, cnt);
        } else {
            if (o.egab[un.x] == FACE_UNSURE) edge_is(un.x, un.i, edge_violated(cd, pp, un.i, un.j));
        }
    }
}
template <int SLOT, bool APEX>
__global__ void __launch_bounds__(AC2_BLOCK, 8) k_ac2(Cands cd, PredParams pp, int what, Ac2Out o, Counters *cnt,
                                                       const int *__restrict__ stop) {
    if (stop && *stop) return;
    __shared__ float4 rows[ac2_rows<SLOT>()];
    ac2_part<SLOT, APEX>(cd, pp, xcd_block(), what, o, cnt, rows);
}

// Tetrahedra of a build. A group's triangles are cut into 2^split slices (one, but
// where few groups have long rows: tet_split); slice v, of group v >> split, has its
// tetrahedra at [at(v), at(v) + num[v]) with at(v) = tet_base[v], or v * cap where
// tet_base is null (slices * cap < 2^31: tet_slab). num: the candidates left to test
// (k_tetrahedra; exact even where the slab is too small, which sets
// Counters::overflow). Once k_tet_ac2 has run, kept[g] of them, in order, are at
// [base(g), base(g) + kept[g]). A tetrahedron is (t, f): its triangle (i, j, k) and its
// edge (i, l).
constexpr int MOST_SLICES = 32;
struct Tets {
    const int *tet_base;
    int cap, split;
    int *t, *t2;  // candidates: triangles (i, j, k) and (i, j, l); t2 becomes f
    double *size;
    int4 *face;   // the facets (sweep only)
    int *num, *kept, *cand, *slice_cand;  // cand: candidates in Sigma_ortho^3 (slice_cand is cand with one slice)
    __device__ __forceinline__ int at(int v) const { return tet_base ? tet_base[v] : v * cap; }
    __device__ __forceinline__ int room(int v) const { return tet_base ? tet_base[v + 1] - tet_base[v] : cap; }
    __device__ __forceinline__ int base(int g) const { return at(g << split); }
};

// A group's candidate tetrahedra: all six edges in Sigma_ortho^1, not flat,
// OrthoSize <= alpha (all six suffice, since OrthoSize grows from face to
// coface, Sec. 4.3). The balls k of TRI_CH triangles (i, j, k) and their edges
// (i, j) are held in LDS. APEX: only those that the triangle's two apex balls do
// not violate are left to test (large radii: one in thirty).
// Bound by waits (half of the time; barriers between the tests and the loads of
// a candidate's other balls), so by the blocks in flight: with 512 triangles
// at a time, 26 KB of LDS and five blocks a CU, 101 us at 3M atoms and alpha = 0
// and 663 at 100,000 with solvent-accessible radii; with 768 triangles, 32 KB and
// four blocks 116 and 779; with 256 113 and 710.
// APEX: a block takes a slice of the group's triangles (Tets), with the later ones of
// their edges as seconds (100 atoms grown by 4 A a build of 480 us, 1,184 with a block
// a group; 289 balls that all meet 4,120, 13,240).
constexpr int TRI_PT = 2, TRI_CH = TRI_PT * BLOCK, TRI_AHEAD = 64;
struct TetLds {
    int4 sk[TRI_CH + TRI_AHEAD];
    int se[TRI_CH + TRI_AHEAD];
    unsigned short own[PAIR_WIN], hit[PAIR_WIN], res[PAIR_WIN];
    int soff[TRI_CH];
    int wtot[2][NWAVE], cands[NWAVE];
};
template <bool APEX>
__device__ __forceinline__ void tetrahedra_group(const Cands &cd, const PredParams &pp, int v,
                                                 const int2 *__restrict__ apex, const Tets &tt, Counters *cnt, TetLds &l) {
    auto &sk = l.sk;
    auto &se = l.se;
    auto &own = l.own;
    auto &hit = l.hit;
    auto &res = l.res;
    auto &soff = l.soff;
    auto &wtot = l.wtot;
    auto &cands = l.cands;
    // the slice's triangles [t0, te); their pairs' second ones reach to t1
    const int split = APEX ? tt.split : 0, g = v >> split, part = v & ((1 << split) - 1);
    const long long tris = cd.tri_cnt[g];
    const int t1 = cd.tri_base[g] + (int)tris;
    const int t0 = cd.tri_base[g] + (int)(tris * part >> split), te = cd.tri_base[g] + (int)(tris * (part + 1) >> split);
    const int w = wave_id(), lane = lane_id();
    const int4 *const atom = cd.atom;
    const int qb = tt.at(v), qcap = tt.room(v);
    int num = 0, nc = 0;
    for (int c0 = t0; c0 < te; c0 += TRI_CH) {
        const int held = min(TRI_CH + TRI_AHEAD, t1 - c0);
#pragma unroll 1
        for (int x = threadIdx.x; x < held; x += BLOCK) {
            sk[x] = atom[cd.up[cd.tri_f[c0 + x]]];
            se[x] = cd.tri_e[c0 + x];
        }
        __syncthreads();
        // later triangles of the same edge
        int later[TRI_PT];
#pragma unroll
        for (int u = 0; u < TRI_PT; u++) {
            const int x = threadIdx.x * TRI_PT + u;
            later[u] = 0;
            if (c0 + x < te) {
                const int e = se[x];
                int y = x + 1;
#pragma unroll 1
                while (c0 + y < t1 && (y < held ? se[y] : cd.tri_e[c0 + y]) == e) y++;
                later[u] = y - x - 1;
            }
        }
        int pairs;
        const int off = pair_scan<TRI_PT>(later, soff, &pairs);
        auto far_ball = [&](int x) { return x < held ? sk[x] : atom[cd.up[cd.tri_f[c0 + x]]]; };
        for (int w0 = 0; w0 < pairs; w0 += PAIR_WIN) {
            pair_owners<TRI_PT>(w0, off, later, own);
            const int wn = min(PAIR_WIN, pairs - w0);
            // second triangle of pair x of the window, less c0 (the first is own[x])
            auto second = [&](int x) { const int o = own[x]; return o + 1 + (w0 + x - soff[o]); };
            const int p1 = part_of(wn);
            const int h = wave_filter(wn, p1, hit, [&](int x, int &v) {
                v = x;
                return spheres_cross(far_ball(own[x]), far_ball(second(x)), pp);
            });
            if (lane == 0) wtot[0][w] = h;
            __syncthreads();
            Parts hs;
            hs.load(wtot[0], p1);
            const int p2 = part_of(hs.total);
            const int r = wave_filter(hs.total, p2, res, [&](int x, int &v) {
                v = hit[hs.slot(x)];
                const int o = own[v], o2 = second(v);
                const int e = se[o];
                const int i = cd.edge_i[e], j = cd.up[e];
                // the apex balls are loaded along with the tetrahedron's
                const int2 q = APEX && !pp.force_exact ? apex[c0 + o] : make_int2(0, 0);
                const int l = APEX ? cd.up[cd.tri_f[c0 + o2]] : 0;
                const int4 vi = atom[i], vj = atom[j];
                const int4 q0 = APEX ? atom[q.x] : vi, q1 = APEX ? atom[q.y] : vi;
                const Tet te = tet_setup(vi, vj, sk[o], far_ball(o2), pp);
                if (te.D == 0) return false;
                const TetFilter tf = tet_filter(te);
                int sg = pp.force_exact ? 0 : tet_ac3_filter(te, pp);
                if (sg == 0) {
                    if (!pp.force_exact) note_fallback(cnt);
                    const int io = opaque(i);
                    sg = tet_ac3_exact(tet_setup(atom[io], atom[j], sk[o], far_ball(o2), pp), pp) ? 1 : -1;
                }
                if (sg < 0) return false;
                nc++;
                if (APEX && !pp.force_exact) {
                    if (q.x != j && q.x != l && tet_violation_filter(tf, q0) < 0) return false;
                    if (q.y != j && q.y != l && tet_violation_filter(tf, q1) < 0) return false;
                }
                return true;
            });
            if (lane == 0) wtot[1][w] = r;
            __syncthreads();
            Parts rs;
            rs.load(wtot[1], p2);
#pragma unroll 1
            for (int x = threadIdx.x; x < rs.total; x += BLOCK) {
                const int v = res[rs.slot(x)];
                const int at = num + x;
                if (at < qcap) {
                    tt.t[qb + at] = c0 + own[v];
                    tt.t2[qb + at] = c0 + second(v);
                } else {
                    cnt->overflow = 1;
                }
            }
            num += rs.total;
            __syncthreads();
        }
        __syncthreads();
    }
    for (int o = WAVE / 2; o > 0; o >>= 1) nc += __shfl_xor(nc, o, WAVE);
    if (lane == 0) cands[w] = nc;
    __syncthreads();
    if (threadIdx.x == 0) {
        tt.num[v] = num;
        int s = 0;
        for (int k = 0; k < NWAVE; k++) s += cands[k];
        tt.slice_cand[v] = s;
    }
}
template <bool APEX>
__global__ void __launch_bounds__(BLOCK, 5) k_tetrahedra(Cands cd, PredParams pp, const int2 *__restrict__ apex, Tets tt,
                                                          Counters *cnt, const int *__restrict__ stop) {
    if (stop && *stop) return;
    __shared__ __align__(16) char lds[sizeof(TetLds)];
    tetrahedra_group<APEX>(cd, pp, xcd_block(), apex, tt, cnt, *reinterpret_cast<TetLds *>(lds));
}

// Both in one launch, the groups' tetrahedra first: neither needs the other
// where no apex balls are used, and up to TET_AC2_BALLS balls each leaves room
// beside it (with the tetrahedra's registers and LDS, four blocks a CU). A build
// of 260 atoms 134 us against 138, 1,003 137 against 142, 16,000 at alpha = 2 224
// against 233; at 50,000 and 100,000 the same within 1 %.
constexpr int TET_AC2_BALLS = 1 << 16;
template <int SLOT>
__global__ void __launch_bounds__(BLOCK, 4) k_tetrahedra_ac2(Cands cd, PredParams pp, int groups, Tets tt, Ac2Out o,
                                                              Counters *cnt, const int *__restrict__ stop) {
    if (stop && *stop) return;
    static_assert(AC2_BLOCK == BLOCK, "one launch");
    constexpr size_t ROWS = ac2_rows<SLOT>() * sizeof(float4);
    __shared__ __align__(16) char lds[sizeof(TetLds) > ROWS ? sizeof(TetLds) : ROWS];
    if ((int)blockIdx.x < groups)
        tetrahedra_group<false>(cd, pp, xcd_block(blockIdx.x, groups), nullptr, tt, cnt, *reinterpret_cast<TetLds *>(lds));
    else
        ac2_part<SLOT, false>(cd, pp, xcd_block(blockIdx.x - groups, gridDim.x - groups), AC2_EDGES | AC2_TRIANGLES, o,
                              cnt, reinterpret_cast<float4 *>(lds));
}

// AC2 of a group's candidate tetrahedra (Step 2): kept iff no ball is strictly
// closer in power to the ortho-centre. The kept ones move to the front of the
// group's range, in order, with their Size, and record themselves on their
// facets (Step 3) unless SWEEP (the candidates of several alpha values, pruned
// per alpha later: tt.face then holds the facets). Blocks of NT threads: one
// wave where a group has some tens of candidates (four times as many groups in
// flight: 139 against 191 us at 3M atoms and alpha = 0), else BLOCK, with half
// the registers for twice the waves (212 against 257 us at 100,000 atoms with
// solvent-accessible radii; the one-wave blocks fit all at once either way). Where
// a group outgrew its slab nothing is tested: all is run again over counted ranges.
// TESTED: after a counted neighbour search k_tet_test has done the walks, with several
// blocks a group (or slice), and here a group's slices come together: a ball with
// thousands of neighbours has thousands of candidates, each with the walk along its row (1,334 small balls around one, all grown: a build
// 20.4 ms by the one block of its group, 6.7 as this).
__global__ void __launch_bounds__(BLOCK, 8) k_tet_test(Cands cd, PredParams pp, Tets tt, Counters *cnt) {
    const int v = xcd_block();  // a slice
    if (cnt->overflow) return;
    const int qb = tt.at(v), num = min(tt.num[v], tt.room(v));
    for (int x = (int)blockIdx.y * BLOCK + (int)threadIdx.x; x < num; x += (int)gridDim.y * BLOCK) {
        const int t = tt.t[qb + x], t2 = tt.t2[qb + x];
        const int e = cd.tri_e[t];
        const int i = cd.edge_i[e], j = cd.up[e], k = cd.up[cd.tri_f[t]], l = cd.up[cd.tri_f[t2]];
        if (!tet_ac2(cd, tet_setup(cd.atom[i], cd.atom[j], cd.atom[k], cd.atom[l], pp), pp, i, j, k, l, cnt))
            tt.t2[qb + x] = ~t2;
    }
}
template <bool SWEEP, int NT, bool TESTED = false>
__global__ void __launch_bounds__(NT, NT == WAVE ? 4 : 8) k_tet_ac2(Cands cd, PredParams pp, const unsigned char *__restrict__ tgab,
                                                       long long *__restrict__ tri_min, Tets tt, Counters *cnt,
                                                       const int *__restrict__ stop) {
    if (stop && *stop) return;
    __shared__ int wtot[2][NT / WAVE];
    const int g = xcd_block();
    if (cnt->overflow) {  // some group outgrew its slab: all run again, over counted ranges
        if (threadIdx.x == 0) tt.kept[g] = 0;
        return;
    }
    const int split = TESTED ? tt.split : 0, v0 = g << split;
    const int qb = tt.at(v0);
    const int w = wave_id(), lane = lane_id();
    // the slices' candidates as one list (a loop over slices of a few candidates each
    // would be a chain of 32 rounds)
    __shared__ int first[TESTED ? MOST_SLICES + 1 : 1];
    int num = 0;
    if constexpr (TESTED) {
        const int m = lane < 1 << split ? min(tt.num[v0 + lane], tt.room(v0 + lane)) : 0;
        const int incl = wave_inclusive_scan(m);
        if (threadIdx.x < MOST_SLICES) first[threadIdx.x + 1] = incl;
        if (threadIdx.x == 0) first[0] = 0;
        if (split > 0) {
            const int c = wave_inclusive_scan(lane < 1 << split ? tt.slice_cand[v0 + lane] : 0);
            if (threadIdx.x == WAVE - 1) tt.cand[g] = c;
        }
        __syncthreads();
        num = first[1 << split];
    } else {
        num = min(tt.num[g], tt.room(g));
    }
    auto place = [&](int x) {
        if (!TESTED) return qb + x;
        int v = 0;
        for (int step = 1 << split >> 1; step > 0; step >>= 1) v += first[v + step] <= x ? step : 0;
        return tt.at(v0 + v) + x - first[v];
    };
    int kept = 0;
    for (int c0 = 0, turn = 0; c0 < num; c0 += NT, turn ^= 1) {
        const int x = c0 + threadIdx.x;
        bool keep = false;
        int t = 0, t2 = 0, f2 = 0;
        if (x < num) {
            const int at = place(x);
            t = tt.t[at];
            t2 = tt.t2[at];
            if constexpr (TESTED) {
                keep = t2 >= 0;
                f2 = cd.tri_f[keep ? t2 : ~t2];
            } else {
                f2 = cd.tri_f[t2];
                const int e = cd.tri_e[t];
                const int i = cd.edge_i[e], j = cd.up[e], k = cd.up[cd.tri_f[t]], l = cd.up[f2];
                const int4 vi = cd.atom[i], vj = cd.atom[j], vk = cd.atom[k], vl = cd.atom[l];
                keep = tet_ac2(cd, tet_setup(vi, vj, vk, vl, pp), pp, i, j, k, l, cnt);
            }
        }
        const unsigned long long mask = __ballot(keep);
        if (lane == 0) wtot[turn][w] = __popcll(mask);
        __syncthreads();  // also: every candidate of the round is read before a kept one is written over it
        int at = kept + __popcll(mask & ((1ull << lane) - 1ull));
#pragma unroll
        for (int u = 0; u < NT / WAVE; u++) {
            if (u < w) at += wtot[turn][u];
            kept += wtot[turn][u];
        }
        if (keep) {
            tt.t[qb + at] = t;
            tt.t2[qb + at] = f2;
            const int e = opaque(cd.tri_e[t]);
            const double sz = tet_size_canon(cd.atom[cd.edge_i[e]], cd.atom[cd.up[e]], cd.atom[cd.up[cd.tri_f[t]]],
                                             cd.atom[cd.up[f2]], pp);
            tt.size[qb + at] = sz;
            const int4 fc = tet_facets(cd, g, t, t2);
            if (SWEEP) {
                tt.face[qb + at] = fc;
            } else {
                const long long key = ordered_from_double(sz);
                mark_face(tgab, tri_min, fc.x, key, cnt);
                mark_face(tgab, tri_min, fc.y, key, cnt);
                mark_face(tgab, tri_min, fc.z, key, cnt);
                mark_face(tgab, tri_min, fc.w, key, cnt);
            }
        }
    }
    if (threadIdx.x == 0) tt.kept[g] = kept;
}

// ---------------------------------------------------------------------------
// Pruning of one alpha: a triangle's or edge's status afterwards is in place of
// its AC2 flag.

// Triangles (Step 3): kept iff AC2 holds at the ortho-centre or a kept
// tetrahedron has it as a facet; Size is then the OrthoSize or the least Size
// of a kept tetrahedron. Kept triangles record themselves on their edges that
// fail AC2; the edge (j, k) is looked up in j's row only if j owns such an edge
// (eng: about one ball in ten at alpha = 0). Counts the kept triangles and
// tetrahedra of every ball.
// LIST: also the kept triangles of the group, in order, at list[tri_base[g] ...]
// (list_cnt[g] of them): for radii of which one candidate in nine is kept, so
// that neither the marks nor the output look at every candidate (k_rows 256 ->
// 117 us at 100,000 atoms with solvent-accessible radii, this 219 -> 102; where
// most are kept the list is only one more array).
template <bool LIST>
__global__ void __launch_bounds__(BLOCK) k_tri_final(Cands cd, unsigned char *__restrict__ tgab,
                                                      const double *__restrict__ tsize,
                                                      const long long *__restrict__ tri_min,
                                                      const unsigned char *__restrict__ egab,
                                                      const unsigned char *__restrict__ eng,
                                                      long long *__restrict__ edge_min, Tets tt,
                                                      int2 *__restrict__ ball_cnt, int *__restrict__ list,
                                                      int *__restrict__ list_cnt, Counters *cnt,
                                                      const int *__restrict__ stop) {
    if (stop && *stop) return;
    __shared__ int tc[GROUP], qc[GROUP], wtot[2][NWAVE];
    const int g = xcd_block();
    const int b0 = g << cd.gshift, nb = min(1 << cd.gshift, cd.n - b0);
    const int w = wave_id(), lane = lane_id();
    tc[threadIdx.x] = qc[threadIdx.x] = 0;
    __syncthreads();
    const int t0 = cd.tri_base[g], t1 = t0 + cd.tri_cnt[g];
    auto is_kept = [&](int t) { return tgab[t] == FACE_GABRIEL || tri_min[t] != ORDERED_POS_INF; };
    auto finish = [&](int t) {  // a kept triangle
        const int e = cd.tri_e[t], f = cd.tri_f[t];
        const bool gab = tgab[t] == FACE_GABRIEL;
        if (!gab) tgab[t] = FACE_ATTACHED;
        const int i = cd.edge_i[e], j = cd.up[e];
        atomicAdd(&tc[i - b0], 1);
        const bool own = eng[i], other = eng[j];
        if (!own && !other) return;
        const long long key = gab ? ordered_from_double(tsize[t]) : tri_min[t];
        if (own) {
            mark_face(egab, edge_min, e, key, cnt);
            mark_face(egab, edge_min, f, key, cnt);
        }
        if (other) mark_face(egab, edge_min, find_edge(cd, j, cd.up_id[f]), key, cnt);
    };
    if (LIST) {
        // the kept ones first, then their marks in full waves
        int kept = 0;
        for (int c0 = t0, turn = 0; c0 < t1; c0 += BLOCK, turn ^= 1) {
            const int t = c0 + threadIdx.x;
            const bool in = t < t1 && is_kept(t);
            const unsigned long long mask = __ballot(in);
            if (lane == 0) wtot[turn][w] = __popcll(mask);
            __syncthreads();
            int at = kept + __popcll(mask & ((1ull << lane) - 1ull));
#pragma unroll
            for (int v = 0; v < NWAVE; v++) {
                if (v < w) at += wtot[turn][v];
                kept += wtot[turn][v];
            }
            if (in) list[t0 + at] = t;
        }
        if (threadIdx.x == 0) list_cnt[g] = kept;
        __syncthreads();
        for (int x = threadIdx.x; x < kept; x += BLOCK) finish(list[t0 + x]);
    } else {
        for (int t = t0 + threadIdx.x; t < t1; t += BLOCK)
            if (is_kept(t)) finish(t);
    }
    const int qb = tt.base(g), qn = tt.kept[g];
    for (int q = threadIdx.x; q < qn; q += BLOCK) atomicAdd(&qc[cd.edge_i[cd.tri_e[tt.t[qb + q]]] - b0], 1);
    __syncthreads();
    if ((int)threadIdx.x < nb) ball_cnt[b0 + threadIdx.x] = make_int2(tc[threadIdx.x], qc[threadIdx.x]);
}

// Output record of a ball at its input id: kept edges, triangles and
// tetrahedra it is the least id of, and in .w its weight W if it passes AC2 at
// its own centre (a vertex of Size -W), VERT_MAYBE if it does not (a vertex iff
// its vert_min is finite), VERT_OUT if -W > alpha.
enum { VERT_OUT = 0, VERT_MAYBE = -1 };

// Edges (Step 4): as triangles; a kept edge records itself on its ends that
// fail AC2 (Step 5; vert_min by input id; cnt->vng: some ball does). A thread
// per ball, over its few edges. Writes the balls' output records: bound by that
// scatter (a line each; 75 us at 3M balls).
__global__ void __launch_bounds__(BLOCK) k_edge_final(Cands cd, PredParams pp, int shortcut,
                                                       unsigned char *__restrict__ egab,
                                                       const long long *__restrict__ edge_min,
                                                       const unsigned char *__restrict__ vgab,
                                                       const unsigned char *__restrict__ eng,
                                                       long long *__restrict__ vert_min,
                                                       const int2 *__restrict__ ball_cnt, int4 *__restrict__ rec,
                                                       const Counters *__restrict__ cnt, const int *__restrict__ stop) {
    if (stop && *stop) return;
    const int s = xcd_block() * BLOCK + threadIdx.x;
    if (s >= cd.n) return;
    const int e0 = cd.up_start[s], e1 = cd.up_start[s + 1];
    const int2 c = ball_cnt[s];
    const int W = cd.atom[s].w, u = cd.perm[s];
    int kept = e1 - e0;
    if (eng[s]) {
        for (int e = e0; e < e1; e++) {
            if (egab[e] == FACE_GABRIEL) continue;
            if (edge_min[e] == ORDERED_POS_INF) kept--;
            else egab[e] = FACE_ATTACHED;
        }
    }
    const bool vs = vgab[s];
    if (cnt->vng) {
        for (int e = e0; e < e1; e++) {
            const int st = egab[e], j = cd.up[e];
            if (st == FACE_OUT) continue;
            const bool vj = vgab[j];
            if (vs && vj) continue;
            const long long key = st == FACE_GABRIEL ? ordered_from_double(edge_size_canon(cd.atom[s], cd.atom[j]))
                                                     : edge_min[e];
            if (!vs) atomicMin(&vert_min[u], key);
            if (!vj) atomicMin(&vert_min[cd.up_id[e]], key);
        }
    }
    const bool ball = (i64)W + pp.aq >= 0;  // OrthoSize -W <= alpha
    rec[u] = make_int4(kept, c.x, c.y, !ball ? VERT_OUT : (shortcut || vs ? W : VERT_MAYBE));
}

}  // namespace acx
