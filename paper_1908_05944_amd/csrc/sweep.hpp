// Alpha sweep (gfx950 device code): the complexes of one ball set for many
// alpha values from the candidates of the largest.
//
// For a candidate simplex the AC3 test "OrthoSize <= alpha" (Sec. 3.1,
// Step 1) is monotone in alpha, so it holds exactly from an integer
// threshold on (alpha in mA^2): the least integer a with OrthoSize <= a. AC2
// (Steps 2-5) does not depend on alpha. The preparation kernels below find
// each candidate's threshold once with the exact predicates and lay every
// per-candidate quantity out in the output order (rows sorted by input ids),
// with face references given as places in that order. The kernels of one
// alpha are then integer comparisons, the attachment of Steps 3-5 and a
// compaction, all streaming over the output order.
#pragma once
#include "emit.hpp"

namespace acx {

// Least integer a in (lo, hi] with ac3(a) true, for an exact test that is
// false at lo and at every a below the threshold, and true at hi and above.
// A float64 estimate of the OrthoSize is corrected by exact tests; bisection
// backs the correction up.
template <class F>
__device__ int entry_threshold(double est, i64 lo, i64 hi, F &&ac3) {
    i64 a = (i64)ceil(est);
    a = a <= lo ? lo + 1 : (a > hi ? hi : a);
    for (int it = 0; it < 4 && a < hi && !ac3(a); it++) a++;
    for (int it = 0; it < 4 && a - 1 > lo && ac3(a - 1); it++) a--;
    if (ac3(a) && (a - 1 <= lo || !ac3(a - 1))) return (int)a;
    i64 l = lo, h = hi;
    while (h - l > 1) {
        const i64 m = l + (h - l) / 2;
        if (ac3(m)) h = m; else l = m;
    }
    return (int)h;
}

constexpr int NO_ENTRY = INT_MAX;  // threshold of a candidate that fails AC2

// Output record of every ball of a sweep: all its candidates, kept at some
// alpha or not (tetrahedra: those that pass AC2; the others are in no K_alpha).
__global__ void __launch_bounds__(BLOCK) k_sweep_counts(Cands cd, Tets tt, int4 *__restrict__ rec) {
    __shared__ int tc[GROUP], qc[GROUP];
    const int g = xcd_block();
    const int b0 = g << cd.gshift, nb = min(1 << cd.gshift, cd.n - b0);
    tc[threadIdx.x] = qc[threadIdx.x] = 0;
    __syncthreads();
    const int t0 = cd.tri_base[g], t1 = t0 + cd.tri_cnt[g];
    for (int t = t0 + threadIdx.x; t < t1; t += BLOCK) atomicAdd(&tc[cd.edge_i[cd.tri_e[t]] - b0], 1);
    const int qb = tt.base(g), qn = tt.kept[g];
    for (int x = threadIdx.x; x < qn; x += BLOCK) atomicAdd(&qc[cd.edge_i[cd.tri_e[tt.t[qb + x]]] - b0], 1);
    __syncthreads();
    const int s = b0 + threadIdx.x;
    if ((int)threadIdx.x < nb)
        rec[cd.perm[s]] = make_int4(cd.up_start[s + 1] - cd.up_start[s], tc[threadIdx.x], qc[threadIdx.x], VERT_OUT);
}

// From the scanned records (base): the place in the output order of candidate
// c of dimension d owned by sorted ball s is adj[s].d + c (d = 1, 2, 3 in .x,
// .y, .z).
__global__ void __launch_bounds__(BLOCK) k_sweep_adj(Cands cd, Tets tt, const int4 *__restrict__ base,
                                                      int4 *__restrict__ adj) {
    const int g = blockIdx.x, s = (g << cd.gshift) + threadIdx.x;
    const bool in = (int)threadIdx.x < (1 << cd.gshift) && s < cd.n;
    const int u = in ? cd.perm[s] : 0;
    const int4 lo = in ? base[u] : make_int4(0, 0, 0, 0), hi = in ? base[u + 1] : lo;
    int tot;
    const int ft = cd.tri_base[g] + block_exclusive_scan<BLOCK>(hi.y - lo.y, &tot);
    const int fq = tt.base(g) + block_exclusive_scan<BLOCK>(hi.z - lo.z, &tot);
    if (in) adj[s] = make_int4(lo.x - cd.up_start[s], lo.y - ft, lo.z - fq, 0);
}

// Edges: threshold, Size and row of every candidate, at its place.
__global__ void __launch_bounds__(BLOCK) k_sweep_prep_edge(Cands cd, int E, const unsigned char *__restrict__ egab,
                                                            const int4 *__restrict__ adj, i64 aq_max,
                                                            int *__restrict__ thr, double *__restrict__ sz,
                                                            int *__restrict__ rows) {
    const int e = xcd_block() * BLOCK + threadIdx.x;
    if (e >= E) return;
    const int i = cd.edge_i[e], j = cd.up[e];
    const int p = adj[i].x + e;
    reinterpret_cast<int2 *>(rows)[p] = make_int2(cd.perm[i], cd.up_id[e]);
    if (!egab[e]) {
        thr[p] = NO_ENTRY;
        return;
    }
    const int4 vi = cd.atom[i], vj = cd.atom[j];
    const Edge ed = edge_setup(vi, vj);
    thr[p] = entry_threshold(edge_orthosize(ed), -(i64)vi.w - 1, aq_max, [&](i64 a) { return edge_ac3(ed, a); });
    sz[p] = edge_size_canon(vi, vj);
}

// Triangles of a group: threshold, Size (the canonical OrthoSize), row, and
// the places of the three edges in the edge output order.
__global__ void __launch_bounds__(BLOCK) k_sweep_prep_tri(Cands cd, const unsigned char *__restrict__ tgab,
                                                           const double *__restrict__ tsize,
                                                           const int4 *__restrict__ adj, PredParams pp,
                                                           int *__restrict__ thr, double *__restrict__ sz,
                                                           int *__restrict__ rows, int4 *__restrict__ face,
                                                           Counters *cnt) {
    const int g = xcd_block();
    const int t0 = cd.tri_base[g], t1 = t0 + cd.tri_cnt[g];
    for (int t = t0 + threadIdx.x; t < t1; t += BLOCK) {
        const int e = cd.tri_e[t], f = cd.tri_f[t];
        const int i = cd.edge_i[e], j = cd.up[e], k = cd.up[f];
        const int4 a = adj[i];
        const int p = a.y + t;
        const int r = find_edge(cd, j, cd.up_id[f]);
        face[p] = make_int4(a.x + e, a.x + f, r < 0 ? -1 : adj[j].x + r, 0);
        rows[3LL * p] = cd.perm[i];
        rows[3LL * p + 1] = cd.up_id[e];
        rows[3LL * p + 2] = cd.up_id[f];
        if (!tgab[t]) {
            thr[p] = NO_ENTRY;
            continue;
        }
        const int4 vi = cd.atom[i], vj = cd.atom[j], vk = cd.atom[k];
        PredParams q = pp;
        thr[p] = entry_threshold(tri_orthosize(tri_setup(vi, vj, vk, pp)), -(i64)vi.w - 1, pp.aq, [&](i64 x) {
            q.aq = x;
            return tri_candidate(vi, vj, vk, q, cnt);
        });
        sz[p] = tsize[t];
    }
}

// Tetrahedra of a group (those that pass AC2): threshold, Size, row, and the
// places of the four facets in the triangle output order.
__global__ void __launch_bounds__(BLOCK) k_sweep_prep_tet(Cands cd, Tets tt, const int4 *__restrict__ adj, PredParams pp,
                                                           int *__restrict__ thr, double *__restrict__ sz,
                                                           int *__restrict__ rows, int4 *__restrict__ face,
                                                           Counters *cnt) {
    const int g = xcd_block();
    const int qb = tt.base(g), qn = tt.kept[g];
    for (int x = qb + threadIdx.x; x < qb + qn; x += BLOCK) {
        const int t = tt.t[x], f2 = tt.t2[x];
        const int e = cd.tri_e[t], f = cd.tri_f[t];
        const int i = cd.edge_i[e], j = cd.up[e];
        const int4 a = adj[i];
        const int p = a.z + x;
        const int4 v0 = cd.atom[i];
        const Tet te = tet_setup(v0, cd.atom[j], cd.atom[cd.up[f]], cd.atom[cd.up[f2]], pp);
        PredParams q = pp;
        thr[p] = entry_threshold(tet_orthosize(te), -(i64)v0.w - 1, pp.aq, [&](i64 y) {
            q.aq = y;
            return tet_ac3(te, q, cnt);
        });
        sz[p] = tt.size[x];
        reinterpret_cast<int4 *>(rows)[p] = make_int4(cd.perm[i], cd.up_id[e], cd.up_id[f], cd.up_id[f2]);
        const int4 fc = tt.face[x];
        face[p] = make_int4(fc.x < 0 ? -1 : a.y + fc.x, fc.y < 0 ? -1 : a.y + fc.y, fc.z < 0 ? -1 : a.y + fc.z,
                            fc.w < 0 ? -1 : adj[j].y + fc.w);
    }
}

// W and whether it passes AC2 at its own centre (or is taken as if), of every
// ball at its input id.
__global__ void __launch_bounds__(BLOCK) k_sweep_prep_vert(Cands cd, const unsigned char *__restrict__ vgab, int shortcut,
                                                            int2 *__restrict__ vert) {
    const int s = xcd_block() * BLOCK + threadIdx.x;
    if (s < cd.n) vert[cd.perm[s]] = make_int2(cd.atom[s].w, shortcut || vgab[s]);
}

// The prepared candidates and the chunk of at most SWEEP_ALPHAS alphas that a
// launch takes (blockIdx.y: the alpha; in launches of their own, 19 an alpha,
// the kernels of 100,000 balls leave the device idle: 495 us for five alphas
// against 217, most of it writes and atomic minima of the kept rows). m[d]: candidates of dimension d, nb[d]: blocks of
// BLOCK of them; mins[d]: m[d] entries an alpha, the least Size of a kept coface
// (order-preserving integer, +inf while none); tsum[d]: nb[d] entries an alpha,
// the kept ones of each block, then their exclusive scan.
constexpr int SWEEP_ALPHAS = 8;
struct Sweep {
    int m[4], nb[4];
    const int2 *vert;
    const int *thr[4];
    const double *sz[4];
    const int *rows[4];
    const int4 *face2, *face3;
    long long *mins[3];
    int *tsum[4];
    i64 aq[SWEEP_ALPHAS];
    Counters *totals[SWEEP_ALPHAS];
    int *out[SWEEP_ALPHAS][4];
    double *out_size[SWEEP_ALPHAS][4];
};

// Whether candidate p of dimension D is in K of alpha a, and its Size in mA^2:
// kept are the candidates that pass AC2 and AC3 (thr <= alpha), and those a
// kept coface recorded itself on.
template <int D>
__device__ __forceinline__ bool sweep_kept(const Sweep &sw, int a, int p, double &size) {
    bool own;
    if constexpr (D == 0) {
        const int2 v = sw.vert[p];
        if ((i64)v.x + sw.aq[a] < 0) return false;
        own = v.y;
        size = -(double)v.x;
    } else {
        own = sw.thr[D][p] <= sw.aq[a];
        if (own) size = sw.sz[D][p];
    }
    if constexpr (D == 3) {
        return own;
    } else {
        if (own) return true;
        const long long mn = sw.mins[D][(long long)a * sw.m[D] + p];
        if (mn == ORDERED_POS_INF) return false;
        size = double_from_ordered(mn);
        return true;
    }
}

// A kept coface records itself on face f unless f passes AC2 (threshold not
// NO_ENTRY: such a face is in K with its own Size whenever a coface is).
__device__ __forceinline__ void sweep_mark(const int *__restrict__ thr, long long *mins, int f, long long key, Counters *cnt) {
    if (f < 0) { atomicOr(&cnt->lookup, 1); return; }
    if (thr[f] != NO_ENTRY) return;
    atomicMin(&mins[f], key);
}

// Candidates of dimension D (3, 2, 1, 0 in turn; Steps 2-5), one thread per row
// of the output order: the kept ones record themselves on their faces and are
// counted by block.
template <int D>
__global__ void __launch_bounds__(BLOCK) k_sweep_mark(Sweep sw, Counters *cnt) {
    const int p = blockIdx.x * BLOCK + threadIdx.x, a = blockIdx.y;
    double size;
    const bool in = p < sw.m[D] && sweep_kept<D>(sw, a, p, size);
    if (D > 0 && in) {
        const long long key = ordered_from_double(size);
        long long *const mins = sw.mins[D - 1] + (long long)a * sw.m[D - 1];
        if constexpr (D == 3) {
            const int4 f = sw.face3[p];
            sweep_mark(sw.thr[2], mins, f.x, key, cnt);
            sweep_mark(sw.thr[2], mins, f.y, key, cnt);
            sweep_mark(sw.thr[2], mins, f.z, key, cnt);
            sweep_mark(sw.thr[2], mins, f.w, key, cnt);
        } else if constexpr (D == 2) {
            const int4 f = sw.face2[p];
            sweep_mark(sw.thr[1], mins, f.x, key, cnt);
            sweep_mark(sw.thr[1], mins, f.y, key, cnt);
            sweep_mark(sw.thr[1], mins, f.z, key, cnt);
        } else if constexpr (D == 1) {
            const int2 v = reinterpret_cast<const int2 *>(sw.rows[1])[p];
            if (!sw.vert[v.x].y) atomicMin(&mins[v.x], key);
            if (!sw.vert[v.y].y) atomicMin(&mins[v.y], key);
        }
    }
    const int kept = __syncthreads_count(in);
    if (threadIdx.x == 0) sw.tsum[D][(long long)a * sw.nb[D] + blockIdx.x] = kept;
}

// Block (d, a): exclusive scan of the blocks' kept counts of dimension d and
// alpha a, and their total.
__global__ void __launch_bounds__(1024) k_sweep_scan(Sweep sw) {
    const int d = blockIdx.x, a = blockIdx.y, nb = sw.nb[d];
    int *const t = sw.tsum[d] + (long long)a * nb;
    int run = 0;
    for (int c0 = 0; c0 < nb; c0 += 1024) {
        const int k = c0 + threadIdx.x;
        const int v = k < nb ? t[k] : 0;
        int tot;
        const int off = block_exclusive_scan<1024>(v, &tot);
        if (k < nb) t[k] = run + off;
        run += tot;
    }
    if (threadIdx.x == 0) {
        Counters *c = sw.totals[a];
        *(d == 0 ? &c->m0 : d == 1 ? &c->m1 : d == 2 ? &c->m2 : &c->m3) = run;
    }
}

// The kept rows of dimension D in output order: block b's first place (scanned
// tsum) plus the place among the block's kept rows.
template <int D>
__device__ __forceinline__ void sweep_write(const Sweep &sw, int b) {
    const int p = b * BLOCK + threadIdx.x, a = blockIdx.y;
    double size;
    const bool in = p < sw.m[D] && sweep_kept<D>(sw, a, p, size);
    int tot;
    const int local = block_exclusive_scan<BLOCK>(in, &tot);
    if (!in) return;
    const long long o = sw.tsum[D][(long long)a * sw.nb[D] + b] + local;
    int *const out = sw.out[a][D];
    if constexpr (D == 0) out[o] = p;
    else if constexpr (D == 1) reinterpret_cast<int2 *>(out)[o] = reinterpret_cast<const int2 *>(sw.rows[D])[p];
    else if constexpr (D == 3) reinterpret_cast<int4 *>(out)[o] = reinterpret_cast<const int4 *>(sw.rows[D])[p];
    else
#pragma unroll
        for (int u = 0; u < 3; u++) out[3 * o + u] = sw.rows[D][3LL * p + u];
    sw.out_size[a][D][o] = size / 1.0e6;  // mA^2 -> A^2
}
__global__ void __launch_bounds__(BLOCK) k_sweep_write(Sweep sw) {
    int b = blockIdx.x;
    if (b < sw.nb[3]) return sweep_write<3>(sw, b);
    b -= sw.nb[3];
    if (b < sw.nb[2]) return sweep_write<2>(sw, b);
    b -= sw.nb[2];
    if (b < sw.nb[1]) return sweep_write<1>(sw, b);
    sweep_write<0>(sw, b - sw.nb[1]);
}

}  // namespace acx
