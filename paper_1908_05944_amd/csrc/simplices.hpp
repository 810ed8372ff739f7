// Candidate triangles and tetrahedra and the pruning (Steps 1-5), for gfx950.
//
// Every simplex belongs to its vertex with the least input id, so the work is
// laid out by ball: a block takes a group of consecutive balls (in sorted order), whose candidate edges are consecutive (upper rows, ordered by
// input id), and enumerates and tests all simplices of those balls. With the
// rows in id order, each ball's simplices come out in output order, so the
// emit needs no sort.
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
// The AC2 tests (long walks along neighbour rows, a thread per simplex) are
// kernels of their own: beside the pair machinery they would hold far more
// registers (194 against 64), and a block's few tetrahedra would wait on its
// triangles.
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
    int n, gshift;
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

// Runs f(q, ball q) over ball i's neighbour row in groups of AC2_GROUP whose
// loads are all issued before the first call, the next group's indices loaded
// while this group is tested. The last group is filled up with `pad`. f
// returns nothing; done() ends the walk after a group.
template <class F, class G>
__device__ __forceinline__ void walk_row(const Cands &cd, int i, int pad, F &&f, G &&done) {
    const int ns = cd.nbr_start[i], ne = ns + cd.nbr_cnt[i];
    int nx[AC2_GROUP];
#pragma unroll
    for (int u = 0; u < AC2_GROUP; u++) nx[u] = cd.nbr[ns + u];  // in bounds: NBR_PAD
    for (int p0 = ns; p0 < ne; p0 += AC2_GROUP) {
        int qs[AC2_GROUP];
        int4 aqs[AC2_GROUP];
#pragma unroll
        for (int u = 0; u < AC2_GROUP; u++) qs[u] = p0 + u < ne ? nx[u] : pad;
        const int pn = p0 + AC2_GROUP < ne ? p0 + AC2_GROUP : p0;  // the last group reloads itself
#pragma unroll
        for (int u = 0; u < AC2_GROUP; u++) nx[u] = cd.nbr[pn + u];
#pragma unroll
        for (int u = 0; u < AC2_GROUP; u++) aqs[u] = cd.atom[qs[u]];
#pragma unroll
        for (int u = 0; u < AC2_GROUP; u++) f(qs[u], aqs[u]);
        if (done()) break;
    }
}

// The AC2 tests below walk the row with the float64 filter alone. Where it
// certified no violator but left some neighbour undecided (exact ties and near
// ties), the row is walked once more with the exact test: inside the first
// walk that code would be there once per neighbour of a group, and the terms
// it needs would be held through the loop (108 registers against 60 for the
// triangles' test).

// AC2 of candidate edge e = (i, j) at its own ortho-centre (Step 4): every
// violator meets the ortho-centre, so it is in i's neighbour row. Writes
// egab[e], and for an edge that fails starts edge_min[e] (the least Size of a
// kept coface) and flags its owner in eng. Every neighbour is tested (no early
// exit: most edges pass, and the loop stays convergent).
__device__ __forceinline__ void edge_ac2(const Cands &cd, const PredParams &pp, int e, int i, int j,
                                         unsigned char *__restrict__ egab, long long *__restrict__ edge_min,
                                         unsigned char *__restrict__ eng) {
    const Edge ed = edge_setup(cd.atom[i], cd.atom[j]);
    bool viol = false, unsure = pp.force_exact;
    if (!pp.force_exact)
        walk_row(cd, i, j, [&](int q, int4 aq) {
            const int sg = edge_violation_filter(ed, aq);
            viol |= (sg < 0) & (q != j);  // padding entries repeat j
            unsure |= (sg == 0) & (q != j);
        }, [] { return false; });
    if (unsure && !viol) {
        const int ns = cd.nbr_start[i], ne = ns + cd.nbr_cnt[i];
#pragma unroll 1
        for (int p = ns; p < ne && !viol; p++) {
            const int q = cd.nbr[p];
            viol = q != j && edge_violation_sign(ed, i, j, cd.atom[q], q, cd.perm, pp.force_exact) < 0;
        }
    }
    egab[e] = (unsigned char)!viol;
    if (viol) {
        edge_min[e] = ORDERED_POS_INF;
        eng[i] = 1;
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

__device__ __forceinline__ double tri_size_canon(int4 a, int4 b, int4 c, const PredParams &pp) {
    int4 v[3] = {a, b, c};
    sort_centres<3>(v);
    return tri_orthosize(tri_setup(v[0], v[1], v[2], pp));
}

__device__ __forceinline__ double tet_size_canon(int4 a, int4 b, int4 c, int4 d, const PredParams &pp) {
    int4 v[4] = {a, b, c, d};
    sort_centres<4>(v);
    return tet_orthosize(tet_setup(v[0], v[1], v[2], v[3], pp));
}

// AC2 of candidate triangle t = (i, j, k) at its own ortho-centre (Step 3;
// violators are in i's neighbour row) and its OrthoSize. Writes tgab[t] and
// tsize[t]. Every neighbour is tested (no early exit, convergent loop).
// APEX: also two neighbours that rule out most tetrahedra on the triangle. The
// ortho-centres of all balls with the triangle lie on its axis, c_t + s n up to
// a scale; ball q, at signed distance D = n.b from the plane, violates a centre
// iff P_q - s D < 0, so on its side of the plane the ball of least P / D (where
// D > 0; of the largest where D < 0) violates every tetrahedron of another
// apex there. The two are found in float32: they are only the first neighbours
// that a candidate is tested against, with the exact predicate.
template <bool APEX>
__device__ __forceinline__ void tri_ac2(const Cands &cd, const PredParams &pp, int t, int i, int j, int k,
                                        unsigned char *__restrict__ tgab, double *__restrict__ tsize,
                                        int2 *__restrict__ apex, Counters *cnt) {
    const int4 vi = cd.atom[i], vj = cd.atom[j], vk = cd.atom[k];
    tsize[t] = tri_size_canon(vi, vj, vk, pp);
    const Tri ts = tri_setup(vi, vj, vk, pp);
    const TriFilter tf = tri_filter(ts);
    const float nx = (float)ts.nx, ny = (float)ts.ny, nz = (float)ts.nz;
    bool viol = false, unsure = pp.force_exact;
    float lo = INFINITY, hi = -INFINITY;
    int qlo = j, qhi = j;  // j: none
    if (!pp.force_exact)
        walk_row(cd, i, j, [&](int q, int4 aq) {
            const bool other = (q != j) & (q != k);
            double P;
            const int sg = tri_violation_filter(tf, aq, P);
            viol |= (sg < 0) & other;
            unsure |= (sg == 0) & other;
            if (APEX) {
                const float D = nx * (float)(aq.x - tf.v0.x) + ny * (float)(aq.y - tf.v0.y) + nz * (float)(aq.z - tf.v0.z);
                const float s = (float)P * __builtin_amdgcn_rcpf(D);
                const bool l = other & (D > 0.0f) & (s < lo), h = other & (D < 0.0f) & (s > hi);
                lo = l ? s : lo;
                qlo = l ? q : qlo;
                hi = h ? s : hi;
                qhi = h ? q : qhi;
            }
        }, [] { return false; });
    if (APEX) apex[t] = make_int2(qlo, qhi);
    if (unsure && !viol) {
        // set up from indices the optimiser cannot follow: nothing of it is
        // kept through the walk above
        const int io = opaque(i);
        const Tri tr = tri_setup(cd.atom[io], cd.atom[j], cd.atom[k], pp);
        const int ns = cd.nbr_start[io], ne = ns + cd.nbr_cnt[io];
#pragma unroll 1
        for (int p = ns; p < ne && !viol; p++) {
            const int q = cd.nbr[p];
            if (q == j || q == k) continue;
            const int4 aq = cd.atom[q];
            double P;
            int sg = pp.force_exact ? 0 : tri_violation_filter(tri_filter(tr), aq, P);
            if (sg == 0) {
                if (!pp.force_exact) note_fallback(cnt);
                sg = tri_violation_exact(tr, i, j, k, aq, q, cd.perm);
            }
            viol = sg < 0;
        }
    }
    tgab[t] = (unsigned char)!viol;
}

// AC2 of tetrahedron (i, j, k, l) against i's neighbour row, ending at the
// first violator (most candidates of large radii fail within a few).
__device__ __forceinline__ bool tet_ac2(const Cands &cd, const TetFilter &tf, const PredParams &pp, int i, int j, int k,
                                        int l, Counters *cnt) {
    bool viol = false, unsure = pp.force_exact;
    if (!pp.force_exact)
        walk_row(cd, i, j, [&](int q, int4 aq) {
            const bool other = (q != j) & (q != k) & (q != l);
            const int sg = tet_violation_filter(tf, aq);
            viol |= (sg < 0) & other;
            unsure |= (sg == 0) & other;
        }, [&] { return viol; });
    if (unsure && !viol) {
        const int io = opaque(i);
        const Tet te = tet_setup(cd.atom[io], cd.atom[j], cd.atom[k], cd.atom[l], pp);
        const int ns = cd.nbr_start[io], ne = ns + cd.nbr_cnt[io];
#pragma unroll 1
        for (int p = ns; p < ne && !viol; p++) {
            const int q = cd.nbr[p];
            if (q == j || q == k || q == l) continue;
            const int4 aq = cd.atom[q];
            int sg = pp.force_exact ? 0 : tet_violation_filter(tet_filter(te), aq);
            if (sg == 0) {
                if (!pp.force_exact) note_fallback(cnt);
                sg = tet_violation_exact(te, i, j, k, l, aq, q, cd.perm);
            }
            viol = sg < 0;
        }
    }
    return !viol;
}

// ---------------------------------------------------------------------------
// AC2 of the candidate edges.
__global__ void __launch_bounds__(BLOCK) k_edge_ac2(Cands cd, const int *__restrict__ E, PredParams pp,
                                                     unsigned char *__restrict__ egab, long long *__restrict__ edge_min,
                                                     unsigned char *__restrict__ eng, const int *__restrict__ stop) {
    if (stop && *stop) return;
    const int e = xcd_block() * BLOCK + threadIdx.x;
    if (e >= *E) return;
    const int i = cd.edge_i[e], j = cd.up[e];
    edge_ac2(cd, pp, e, i, j, egab, edge_min, eng);
}

// Candidate triangles (Sec. 4.3) of a group's edges. The balls of EDGE_CH
// edges' other ends (and of the next EDGE_AHEAD, where a row goes on) are held
// in LDS, so that the pair tests wait for no memory. COUNT: the groups' totals
// only (the first pass of a counted build).
constexpr int EDGE_PT = 2, EDGE_CH = EDGE_PT * BLOCK, EDGE_AHEAD = 64;
template <bool COUNT>
__global__ void __launch_bounds__(BLOCK) k_triangles(Cands cd, PredParams pp, long long *__restrict__ tri_min, Counters *cnt,
                                                      const int *__restrict__ stop) {
    if (stop && *stop) return;
    __shared__ int4 sat[EDGE_CH + EDGE_AHEAD];
    __shared__ unsigned short own[PAIR_WIN], hit[PAIR_WIN], res[PAIR_WIN];
    __shared__ int soff[EDGE_CH];
    __shared__ int wtot[2][NWAVE];
    const int g = xcd_block();
    const int b0 = g << cd.gshift, b1 = min(b0 + (1 << cd.gshift), cd.n);
    const int e0 = cd.up_start[b0], e1 = cd.up_start[b1];
    const int w = wave_id(), lane = lane_id();
    int out = COUNT ? 0 : cd.tri_base[g];
    const int out0 = out;
    for (int c0 = e0; c0 < e1; c0 += EDGE_CH) {
        for (int x = threadIdx.x; x < min(EDGE_CH + EDGE_AHEAD, e1 - c0); x += BLOCK) sat[x] = cd.atom[cd.up[c0 + x]];
        int later[EDGE_PT];
#pragma unroll
        for (int u = 0; u < EDGE_PT; u++) {
            const int e = c0 + threadIdx.x * EDGE_PT + u;
            later[u] = e < e1 ? cd.up_start[cd.edge_i[e] + 1] - e - 1 : 0;
        }
        int pairs;
        const int off = pair_scan<EDGE_PT>(later, soff, &pairs);
        int prev = -1;  // edge (less c0) of the last triangle of the windows before
        // the ball at the far end of edge c0 + x
        auto far_ball = [&](int x) { return x < EDGE_CH + EDGE_AHEAD ? sat[x] : cd.atom[cd.up[c0 + x]]; };
        for (int w0 = 0; w0 < pairs; w0 += PAIR_WIN) {
            pair_owners<EDGE_PT>(w0, off, later, own);
            const int wn = min(PAIR_WIN, pairs - w0);
            // second edge of pair x of the window, less c0 (the first is own[x])
            auto second = [&](int x) { const int o = own[x]; return o + 1 + (w0 + x - soff[o]); };
            // pairs of the upper row whose spheres cross
            const int p1 = part_of(wn);
            const int h = wave_filter(wn, p1, hit, [&](int x, int &v) {
                v = x;
                return spheres_cross(far_ball(own[x]), far_ball(second(x)), pp);
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
                    // in the window of its first)
                    const bool first = x > 0 ? own[res[rs.slot(x - 1)]] != o : prev != o;
                    if (first) cd.tri_first[c0 + o] = out + x;
                }
            }
            if (rs.total > 0) prev = own[res[rs.slot(rs.total - 1)]];
            out += rs.total;
            __syncthreads();
        }
        __syncthreads();  // sat and soff are rewritten by the next round
    }
    if (threadIdx.x == 0) cd.tri_cnt[g] = out - out0;
}

// ---------------------------------------------------------------------------
// A face that passes AC2 itself is in K with Size = OrthoSize whatever its
// cofaces do, so only faces failing AC2 record the kept coface: the least
// Size of their kept cofaces (order-preserving integer; +inf while none), so
// such a face is kept iff that minimum is finite.
// gab: the faces' status.
enum { FACE_OUT = 0, FACE_GABRIEL = 1, FACE_ATTACHED = 2 };  // AC2 leaves 0 or 1
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

// AC2 and OrthoSize of a group's candidate triangles. Eight waves per SIMD: the
// walk along the neighbour row needs less than 64 registers, what is spilled
// belongs to the exact test.
template <bool APEX>
__global__ void __launch_bounds__(BLOCK, 8) k_tri_ac2(Cands cd, PredParams pp, unsigned char *__restrict__ tgab,
                                                       double *__restrict__ tsize, int2 *__restrict__ apex,
                                                       Counters *cnt, const int *__restrict__ stop) {
    if (stop && *stop) return;
    const int g = xcd_block();
    const int t0 = cd.tri_base[g], t1 = t0 + cd.tri_cnt[g];
    for (int t = t0 + threadIdx.x; t < t1; t += BLOCK) {
        const int e = cd.tri_e[t];
        const int i = cd.edge_i[e], j = cd.up[e], k = cd.up[cd.tri_f[t]];
        tri_ac2<APEX>(cd, pp, t, i, j, k, tgab, tsize, apex, cnt);
    }
}

// Tetrahedra of a build: group g's are at [base, base + num[g]) with base =
// tet_base[g], or g * cap where tet_base is null. num: first the candidates
// left to test (k_tetrahedra; exact even where the slab is too small, which sets
// Counters::overflow), and kept[g] of them, in order, once k_tet_ac2 has run.
// A tetrahedron is (t, f): its triangle (i, j, k) and its edge (i, l).
struct Tets {
    const int *tet_base;
    int cap;
    int *t, *t2;  // candidates: triangles (i, j, k) and (i, j, l); t2 becomes f
    double *size;
    int4 *face;   // the facets (sweep only)
    int *num, *kept, *cand;  // cand: candidates in Sigma_ortho^3
    __device__ __forceinline__ int base(int g) const { return tet_base ? tet_base[g] : g * cap; }
    __device__ __forceinline__ int room(int g) const { return tet_base ? tet_base[g + 1] - tet_base[g] : cap; }
};

// A group's candidate tetrahedra: all six edges in Sigma_ortho^1, not flat,
// OrthoSize <= alpha (all six suffice, since OrthoSize grows from face to
// coface, Sec. 4.3). The balls k of TRI_CH triangles (i, j, k) and their edges
// (i, j) are held in LDS. APEX: only those that the triangle's two apex balls do
// not violate are left to test (large radii: one in thirty).
constexpr int TRI_PT = 3, TRI_CH = TRI_PT * BLOCK, TRI_AHEAD = 64;
template <bool APEX>
__global__ void __launch_bounds__(BLOCK, 4) k_tetrahedra(Cands cd, PredParams pp, const int2 *__restrict__ apex, Tets tt,
                                                          Counters *cnt, const int *__restrict__ stop) {
    if (stop && *stop) return;
    __shared__ int4 sk[TRI_CH + TRI_AHEAD];
    __shared__ int se[TRI_CH + TRI_AHEAD];
    __shared__ unsigned short own[PAIR_WIN], hit[PAIR_WIN], res[PAIR_WIN];
    __shared__ int soff[TRI_CH];
    __shared__ int wtot[2][NWAVE], cands[NWAVE];
    const int g = xcd_block();
    const int t0 = cd.tri_base[g], t1 = t0 + cd.tri_cnt[g];
    const int w = wave_id(), lane = lane_id();
    const int4 *const atom = cd.atom;
    const int qb = tt.base(g), qcap = tt.room(g);
    int num = 0, nc = 0;
    for (int c0 = t0; c0 < t1; c0 += TRI_CH) {
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
            if (c0 + x < t1) {
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
                const Tet te = tet_setup(atom[i], atom[j], sk[o], far_ball(o2), pp);
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
                    const int2 q = apex[c0 + o];
                    const int l = cd.up[cd.tri_f[c0 + o2]];
                    if (q.x != j && q.x != l && tet_violation_filter(tf, atom[q.x]) < 0) return false;
                    if (q.y != j && q.y != l && tet_violation_filter(tf, atom[q.y]) < 0) return false;
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
        tt.num[g] = num;
        int s = 0;
        for (int k = 0; k < NWAVE; k++) s += cands[k];
        tt.cand[g] = s;
    }
}

// AC2 of a group's candidate tetrahedra (Step 2): kept iff no ball is strictly
// closer in power to the ortho-centre. The kept ones move to the front of the
// group's range, in order, with their Size, and record themselves on their
// facets (Step 3) unless SWEEP (the candidates of several alpha values, pruned
// per alpha later: tt.face then holds the facets). Blocks of NT threads: one
// wave where a group has some tens of candidates (four times as many groups in
// flight: 139 against 191 us at 3M atoms and alpha = 0), else BLOCK.
template <bool SWEEP, int NT>
__global__ void __launch_bounds__(NT, 4) k_tet_ac2(Cands cd, PredParams pp, const unsigned char *__restrict__ tgab,
                                                       long long *__restrict__ tri_min, Tets tt, Counters *cnt,
                                                       const int *__restrict__ stop) {
    if (stop && *stop) return;
    __shared__ int wtot[2][NT / WAVE];
    const int g = xcd_block();
    const int qb = tt.base(g), num = min(tt.num[g], tt.room(g));
    const int w = wave_id(), lane = lane_id();
    int kept = 0;
    for (int c0 = 0, turn = 0; c0 < num; c0 += NT, turn ^= 1) {
        const int x = c0 + threadIdx.x;
        bool keep = false;
        int t = 0, t2 = 0, f2 = 0;
        if (x < num) {
            t = tt.t[qb + x];
            t2 = tt.t2[qb + x];
            f2 = cd.tri_f[t2];
            const int e = cd.tri_e[t];
            const int i = cd.edge_i[e], j = cd.up[e], k = cd.up[cd.tri_f[t]], l = cd.up[f2];
            const int4 vi = cd.atom[i], vj = cd.atom[j], vk = cd.atom[k], vl = cd.atom[l];
            keep = tet_ac2(cd, tet_filter(tet_setup(vi, vj, vk, vl, pp)), pp, i, j, k, l, cnt);
        }
        const unsigned long long mask = __ballot(keep);
        if (lane == 0) wtot[turn][w] = __popcll(mask);
        __syncthreads();  // also: every candidate of the round is read before a kept one is written over it
        int at = kept + __popcll(mask & ((1ull << lane) - 1ull));
#pragma unroll
        for (int v = 0; v < NT / WAVE; v++) {
            if (v < w) at += wtot[turn][v];
            kept += wtot[turn][v];
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
__global__ void __launch_bounds__(BLOCK) k_tri_final(Cands cd, unsigned char *__restrict__ tgab,
                                                      const double *__restrict__ tsize,
                                                      const long long *__restrict__ tri_min,
                                                      const unsigned char *__restrict__ egab,
                                                      const unsigned char *__restrict__ eng,
                                                      long long *__restrict__ edge_min, Tets tt,
                                                      int2 *__restrict__ ball_cnt, Counters *cnt,
                                                      const int *__restrict__ stop) {
    if (stop && *stop) return;
    __shared__ int tc[GROUP], qc[GROUP];
    const int g = xcd_block();
    const int b0 = g << cd.gshift, nb = min(1 << cd.gshift, cd.n - b0);
    tc[threadIdx.x] = qc[threadIdx.x] = 0;
    __syncthreads();
    const int t0 = cd.tri_base[g], t1 = t0 + cd.tri_cnt[g];
    for (int t = t0 + threadIdx.x; t < t1; t += BLOCK) {
        const int e = cd.tri_e[t], f = cd.tri_f[t];
        const bool gab = tgab[t] == FACE_GABRIEL;
        const long long mn = gab ? ORDERED_POS_INF : tri_min[t];
        if (!gab && mn == ORDERED_POS_INF) continue;
        if (!gab) tgab[t] = FACE_ATTACHED;
        const int i = cd.edge_i[e], j = cd.up[e];
        atomicAdd(&tc[i - b0], 1);
        const bool own = eng[i], other = eng[j];
        if (!own && !other) continue;
        const long long key = gab ? ordered_from_double(tsize[t]) : mn;
        if (own) {
            mark_face(egab, edge_min, e, key, cnt);
            mark_face(egab, edge_min, f, key, cnt);
        }
        if (other) mark_face(egab, edge_min, find_edge(cd, j, cd.up_id[f]), key, cnt);
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
// per ball, over its few edges. Writes the balls' output records.
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
