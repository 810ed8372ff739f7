// Volume and boundary area of the union of the balls, from the alpha complex
// at alpha = 0, and their gradients (the complex held fixed).
//
// The union's measure is the alternating sum, over the simplices of the dual
// complex, of the measure of the intersection of their balls (the short
// inclusion-exclusion of Edelsbrunner, 1995); the paper names volume and area
// as what the alpha complex of a molecule is for (Sec. 1). Per simplex of k
// balls, with I the intersection:
//   vol(I)  = (1/3) [ sum_i r_i |P_i| - sum_{i<j} d_ij |F_ij| ]
// where P_i is the patch of sphere i on the boundary of I and F_ij the flat
// face of I on the radical plane of i and j once I is split by the farthest-
// power diagram of its balls (each piece coned from its own centre).
//   |P_i|  = r_i^2 (2 pi - sum of exterior corner angles) - r_i sum_j t_ij phi_ij
// by Gauss-Bonnet, t_ij being the signed distance from centre i to the plane
// and phi_ij the central angle of the boundary arc on the circle S_i & S_j.
// Gradients: d vol / d r_i = |P_i|; d vol / d p_i = sum_j |F_ij| u_ij; the
// boundary area moves by (2 / r_i) times the patch's (vector) area plus
// cot(psi/2) times the length (or int n ds) of each boundary arc of P_i, psi
// the interior dihedral angle of I there.
//
// One thread per corner of a simplex; float64 throughout. The coordinates are the
// caller's float64 ones (not the quantised values the complex was built
// from), so square roots and arc cosines are clamped to their domain.
#pragma once
#include "common.hpp"
#include "radix.hpp"
#include "rules.hpp"

namespace acx {

struct D3 {
    double x, y, z;
};
__device__ __forceinline__ D3 d3(double x, double y, double z) { return D3{x, y, z}; }
__device__ __forceinline__ D3 operator+(D3 a, D3 b) { return d3(a.x + b.x, a.y + b.y, a.z + b.z); }
__device__ __forceinline__ D3 operator-(D3 a, D3 b) { return d3(a.x - b.x, a.y - b.y, a.z - b.z); }
__device__ __forceinline__ D3 operator*(double s, D3 a) { return d3(s * a.x, s * a.y, s * a.z); }
__device__ __forceinline__ double dot(D3 a, D3 b) { return a.x * b.x + a.y * b.y + a.z * b.z; }
__device__ __forceinline__ D3 cross(D3 a, D3 b) {
    return d3(a.y * b.z - a.z * b.y, a.z * b.x - a.x * b.z, a.x * b.y - a.y * b.x);
}
__device__ __forceinline__ D3 unit(D3 a) {
    const double n = sqrt(dot(a, a));
    return n > 0 ? (1.0 / n) * a : a;
}
__device__ __forceinline__ double clamp1(double x) { return fmin(1.0, fmax(-1.0, x)); }

constexpr double PI = 3.14159265358979323846;

// Terms of corner c (ball c) of one simplex of K balls: what the patch P_c
// and the faces and arcs around it contribute. Summed over the corners:
// vol is the intersection's volume (each flat face's d |F| is split evenly
// between its two balls) and area the boundary area. The arc terms are
// computed only if GRAD.
struct CornerTerms {
    double vol;      // (1/3) [r_c |P_c| - 1/2 sum_b d_cb |F_cb|]
    double area;     // |P_c|
    D3 vec;          // vector area of P_c: sum_b |F_cb| u_cb
    double arc_len;  // sum over the arcs of P_c of cot(psi/2) * length
    D3 arc_vec;      // sum over the arcs of P_c of cot(psi/2) * int n_c ds
};

// Exterior angle at corner v of the patch on sphere (p, r) between the arcs
// cut by the planes with normals ua and ub.
__device__ __forceinline__ double corner_angle(D3 v, D3 p, double r, D3 ua, D3 ub) {
    const D3 n = (1.0 / r) * (v - p);
    const D3 ga = unit(ua - dot(ua, n) * n);
    const D3 gb = unit(ub - dot(ub, n) * n);
    return acos(clamp1(dot(ga, gb)));
}

// Vertex of the intersection of 4 balls on the power line of the triple
// opposite ball f: the triple point inside ball f. c is the ortho-centre.
__device__ __forceinline__ D3 triple_vertex(const D3 *P, int f, D3 c, double rho2) {
    const int t0 = f == 0 ? 1 : 0, t1 = f <= 1 ? 2 : 1, t2 = f == 3 ? 2 : 3;  // the balls other than f, ascending
    D3 nt = unit(cross(P[t1] - P[t0], P[t2] - P[t0]));
    if (dot(nt, P[f] - P[t0]) < 0) nt = -1.0 * nt;
    const double beta = dot(nt, c - P[t0]);
    const double tau = -beta + sqrt(fmax(beta * beta + rho2, 0.0));
    return c + tau * nt;
}

// The corner is ball 0: callers rotate the simplex's balls so that every
// index below is a compile-time constant (no scratch arrays).
template <int K, bool GRAD>
__device__ void corner_terms(const D3 *P, const double *R, CornerTerms &o) {
    constexpr int cc = 0;
    o.vec = d3(0, 0, 0);
    o.arc_len = 0;
    o.arc_vec = d3(0, 0, 0);
    if (K == 1) {
        o.vol = 4.0 / 3.0 * PI * R[0] * R[0] * R[0];
        o.area = 4.0 * PI * R[0] * R[0];
        return;
    }
    // point of equal power (in the plane of the centres when K = 3) and rho^2
    D3 c = P[0];
    double rho2 = 0;
    if (K >= 3) {
        const D3 e1 = P[1] - P[0], e2 = P[2] - P[0];
        const double h1 = 0.5 * (dot(e1, e1) - R[1] * R[1] + R[0] * R[0]);
        const double h2 = 0.5 * (dot(e2, e2) - R[2] * R[2] + R[0] * R[0]);
        D3 z;
        if (K == 3) {
            const double g11 = dot(e1, e1), g12 = dot(e1, e2), g22 = dot(e2, e2);
            const double det = g11 * g22 - g12 * g12;
            const double l1 = (h1 * g22 - h2 * g12) / det, l2 = (h2 * g11 - h1 * g12) / det;
            z = l1 * e1 + l2 * e2;
        } else {
            const D3 e3 = P[3] - P[0];
            const double h3 = 0.5 * (dot(e3, e3) - R[3] * R[3] + R[0] * R[0]);
            const D3 c23 = cross(e2, e3), c31 = cross(e3, e1), c12 = cross(e1, e2);
            z = (1.0 / dot(e1, c23)) * (h1 * c23 + h2 * c31 + h3 * c12);
        }
        c = P[0] + z;
        rho2 = R[0] * R[0] - dot(z, z);
    }
    const double rho = sqrt(fmax(rho2, 0.0));
    // K = 4: the triple points the corner's patch and arcs need (triples
    // containing ball 0), indexed by the ball opposite the triple
    D3 tv[4];
    if (K == 4) {
#pragma unroll
        for (int f = 1; f < 4; f++) tv[f] = triple_vertex(P, f, c, rho2);
    }
    const double rc = R[cc];
    double turn = 0, flat = 0, corner = 0;
#pragma unroll
    for (int b = 1; b < K; b++) {
        const D3 dv = P[b] - P[cc];
        const double d = sqrt(dot(dv, dv));
        const D3 u = (1.0 / d) * dv;
        const double tc = (d * d + rc * rc - R[b] * R[b]) / (2 * d);  // centre c to the plane, towards b
        const D3 oc = P[cc] + tc * u;                                  // centre of the circle S_c & S_b
        const double a2 = fmax(rc * rc - tc * tc, 0.0);
        const double rad = sqrt(a2);
        double phi, face;
        D3 mid = d3(0, 0, 0);
        if (K == 2) {
            phi = 2 * PI;
            face = PI * a2;
        } else if (K == 3) {
            const int e = 3 - cc - b;
            const D3 w = unit((P[e] - P[cc]) - dot(P[e] - P[cc], u) * u);
            const double sw = dot(c - oc, w);
            const double half = rad > 0 ? acos(clamp1(sw / rad)) : 0.0;
            face = a2 * half - sw * sqrt(fmax(a2 - sw * sw, 0.0));
            phi = 2 * half;
            mid = w;
        } else {
            // the other two balls e < f
            const int e = b == 1 ? 2 : 1, f = b == 3 ? 2 : 3;
            // the arc runs between the triple points of (c, b, e) and (c, b, f)
            const D3 q1 = tv[f], q2 = tv[e];
            D3 axis = u;
            if (dot(cross(q1 - c, q2 - c), u) < 0) axis = -1.0 * u;
            const D3 r1 = q1 - oc, r2 = q2 - oc;
            double ang = atan2(dot(cross(r1, r2), axis), dot(r1, r2));
            if (ang < 0) ang += 2 * PI;
            phi = rad > 0 ? ang : 0.0;
            face = 0.5 * (a2 * phi + dot(cross(oc - c, q2 - q1), axis));
            const D3 e1 = unit(r1);
            mid = cos(0.5 * phi) * e1 + sin(0.5 * phi) * cross(axis, e1);
        }
        flat += d * face;
        turn += tc * phi;
        o.vec = o.vec + face * u;
        if (GRAD) {
            const double cos_psi = -(rc * rc + R[b] * R[b] - d * d) / (2 * rc * R[b]);
            const double cot_half = sqrt(fmax(1 + cos_psi, 0.0) / fmax(1 - cos_psi, 1e-300));
            const double len = rad * phi;
            o.arc_len += cot_half * len;
            const D3 radial = (a2 * 2 * sin(0.5 * phi)) * mid;  // int (x - o) ds over the arc
            o.arc_vec = o.arc_vec + (cot_half / rc) * ((tc * len) * u + radial);
        }
    }
    // exterior angles at the corners of P_c
    if (K == 3) {
        const D3 nrm = unit(cross(P[1] - P[0], P[2] - P[0]));
        constexpr int j = 1, l = 2;
        const D3 uj = unit(P[j] - P[cc]), ul = unit(P[l] - P[cc]);
        corner = corner_angle(c + rho * nrm, P[cc], rc, uj, ul) + corner_angle(c - rho * nrm, P[cc], rc, uj, ul);
    }
    if (K == 4) {
#pragma unroll
        for (int f = 1; f < 4; f++) {
            const int j = f == 1 ? 2 : 1, l = f == 3 ? 2 : 3;  // the balls other than 0 and f
            corner += corner_angle(tv[f], P[cc], rc, unit(P[j] - P[cc]), unit(P[l] - P[cc]));
        }
    }
    o.area = rc * rc * (2 * PI - corner) - rc * turn;
    o.vol = (rc * o.area - 0.5 * flat) / 3.0;
}

// Balls of simplex s, rotated so that corner c comes first.
template <int K>
__device__ __forceinline__ void load_balls(const int *__restrict__ simp, long long s, int c0,
                                           const double *__restrict__ xyz, const double *__restrict__ rad, D3 *P,
                                           double *R) {
#pragma unroll
    for (int c = 0; c < K; c++) {
        const int id = simp[s * K + (c0 + c) % K];
        const double *p = xyz + 3LL * id;
        P[c] = d3(p[0], p[1], p[2]);
        R[c] = rad[id];
    }
}

constexpr int MEASURE_BLOCK = 256;

// Simplices of a complex by dimension (rows simp[d], count[d] of them), the
// blocks of a launch per dimension, and where a dimension's corners start among
// all (slot of corner k of simplex s of dimension d: first[d] + s (d + 1) + k)
// and its blocks among the blocks of all dimensions.
struct Simplices {
    const int *simp[4];
    long long count[4], first[4];
    int blocks[4], block0[4];
};

// Block b of dimension K - 1, one thread per (simplex, corner) (thread t:
// simplex t / K, corner t % K).
// GRAD: the corner's contribution gV d(V)/d(p, r) + gA d(A)/d(p, r) to its ball,
// as (x, y, z, r), at its slot of contrib, with (gV, gA) = (g[0], g[1]) read
// from device memory. VA: the signed sums of the block's volume and patch-area
// parts at part[2 * block] and part[2 * block + 1].
template <int K, bool VA, bool GRAD>
__device__ __forceinline__ void measure_block(const Simplices &sx, int b, const double *__restrict__ xyz,
                                              const double *__restrict__ rad, const double *__restrict__ g,
                                              double4 *__restrict__ contrib, double *__restrict__ part) {
    const long long t = (long long)b * MEASURE_BLOCK + threadIdx.x;
    const double sg = ((K - 1) & 1) ? -1.0 : 1.0;
    double v = 0, a = 0;
    if (t < sx.count[K - 1] * K) {
        D3 P[K];
        double R[K];
        load_balls<K>(sx.simp[K - 1], t / K, (int)(t % K), xyz, rad, P, R);
        CornerTerms ct;
        corner_terms<K, GRAD>(P, R, ct);
        if (GRAD) {
            const double gV = g[0], gA = g[1];
            const double ir = 2.0 / R[0];
            const D3 gx = (sg * gV) * ct.vec + (sg * gA) * (ir * ct.vec + ct.arc_vec);
            const double gr = sg * (gV * ct.area + gA * (ir * ct.area + ct.arc_len));
            contrib[sx.first[K - 1] + t] = make_double4(gx.x, gx.y, gx.z, gr);
        }
        v = sg * ct.vol;
        a = sg * ct.area;
    }
    if (!VA) return;
    __shared__ double sv[MEASURE_BLOCK / WAVE], sa[MEASURE_BLOCK / WAVE];
    for (int off = WAVE / 2; off > 0; off >>= 1) {
        v += __shfl_down(v, off, WAVE);
        a += __shfl_down(a, off, WAVE);
    }
    const int w = threadIdx.x / WAVE;
    if (lane_id() == 0) {
        sv[w] = v;
        sa[w] = a;
    }
    __syncthreads();
    if (threadIdx.x == 0) {
        double tv = 0, ta = 0;
        for (int k = 0; k < MEASURE_BLOCK / WAVE; k++) {
            tv += sv[k];
            ta += sa[k];
        }
        part[2LL * (sx.block0[K - 1] + b)] = tv;
        part[2LL * (sx.block0[K - 1] + b) + 1] = ta;
    }
}

// All dimensions in one launch, the largest simplices (the longest blocks)
// first. Bound by the float64 chains of the tetrahedra's and triangles' corners
// (square roots, arc cosines), so that it does not matter that points and edges
// run with the tetrahedra's registers (240 a lane with GRAD, two waves per
// SIMD). Fused call, one launch a dimension 43 us at 4,001 balls, this 14; with
// points and edges in a launch of their own 17.4 (25.5 against 22.2 at 16,000,
// 76.9 against 76.1 at 100,000, 145 against 147 at 200,000).
template <bool VA, bool GRAD>
__global__ void __launch_bounds__(MEASURE_BLOCK) k_measure(Simplices sx, const double *__restrict__ xyz,
                                                            const double *__restrict__ rad, const double *__restrict__ g,
                                                            double4 *__restrict__ contrib, double *__restrict__ part) {
    int b = blockIdx.x;
    if (b < sx.blocks[3]) return measure_block<4, VA, GRAD>(sx, b, xyz, rad, g, contrib, part);
    b -= sx.blocks[3];
    if (b < sx.blocks[2]) return measure_block<3, VA, GRAD>(sx, b, xyz, rad, g, contrib, part);
    b -= sx.blocks[2];
    if (b < sx.blocks[1]) return measure_block<2, VA, GRAD>(sx, b, xyz, rad, g, contrib, part);
    measure_block<1, VA, GRAD>(sx, b - sx.blocks[1], xyz, rad, g, contrib, part);
}

// V, A from the nb blocks' parts, summed in a fixed order by one block.
__device__ __forceinline__ void measure_total(const double *__restrict__ part, int nb, double *__restrict__ out) {
    __shared__ double sv[MEASURE_BLOCK / WAVE], sa[MEASURE_BLOCK / WAVE];
    double v = 0, a = 0;
    const double2 *p = reinterpret_cast<const double2 *>(part);
#pragma unroll 4
    for (int b = threadIdx.x; b < nb; b += MEASURE_BLOCK) {
        const double2 x = p[b];
        v += x.x;
        a += x.y;
    }
    for (int off = WAVE / 2; off > 0; off >>= 1) {
        v += __shfl_down(v, off, WAVE);
        a += __shfl_down(a, off, WAVE);
    }
    const int w = threadIdx.x / WAVE;
    if (lane_id() == 0) {
        sv[w] = v;
        sa[w] = a;
    }
    __syncthreads();
    if (threadIdx.x == 0) {
        double tv = 0, ta = 0;
        for (int k = 0; k < MEASURE_BLOCK / WAVE; k++) {
            tv += sv[k];
            ta += sa[k];
        }
        out[0] = tv;
        out[1] = ta;
    }
}
__global__ void __launch_bounds__(MEASURE_BLOCK) k_measure_total(const double *__restrict__ part, int nb,
                                                                  double *__restrict__ out) {
    measure_total(part, nb, out);
}

// ---------------------------------------------------------------------------
// The corners of all simplices sorted by ball (slots ascending within a ball),
// once per complex: radix passes over the key bits above a bucket of 2^shift
// balls, then k_inc_finish orders each bucket on the low bits.

// Ball of every corner slot, and the histogram of the first digit.
__global__ void __launch_bounds__(RS_BLOCK) k_inc_hist(Simplices sx, int M, unsigned *__restrict__ key, int shift,
                                                        int *__restrict__ hist, int tiles) {
    __shared__ int h[RS_BINS];
    h[threadIdx.x] = 0;
    __syncthreads();
    const int base = blockIdx.x * RS_TILE;
#pragma unroll
    for (int r = 0; r < RS_IPT; r++) {
        const int i = base + r * RS_BLOCK + (int)threadIdx.x;
        if (i >= M) break;
        const int d = (i >= sx.first[1]) + (i >= sx.first[2]) + (i >= sx.first[3]);
        const int *p = d == 0 ? sx.simp[0] : d == 1 ? sx.simp[1] : d == 2 ? sx.simp[2] : sx.simp[3];
        const long long f = d == 0 ? 0 : d == 1 ? sx.first[1] : d == 2 ? sx.first[2] : sx.first[3];
        const unsigned k = (unsigned)p[i - f];
        key[i] = k;
        atomicAdd(&h[(k >> shift) & (RS_BINS - 1)], 1);
    }
    __syncthreads();
    hist[rs_hist_at(threadIdx.x, blockIdx.x, tiles)] = h[threadIdx.x];
}

// One bucket per block: its rows [start[b], start[b + 1]) of (key, slot), in
// slot order, are ordered by ball, stably: each wave takes a contiguous part and
// ranks its rows among equal balls with ballots and counters of its own, a
// scan over (ball, wave) places them. No limit on the rows of a bucket or ball.
// At 100,000 balls (196 buckets of some 7,000 rows) 18 us, with 256 threads a
// block 44; three full radix passes and a search for every ball's start, which
// this replaces, took 150.
constexpr int INC_BLOCK = 1024;
__global__ void __launch_bounds__(INC_BLOCK) k_inc_finish(const unsigned *__restrict__ key, const unsigned *__restrict__ pay,
                                                     const int *__restrict__ start, int M, int shift, int n,
                                                     int *__restrict__ inc_start, int *__restrict__ inc_slot) {
    constexpr int NW = INC_BLOCK / WAVE;
    static_assert(INC_KEYS <= INC_BLOCK, "a ball per thread");
    __shared__ int cnt[NW][INC_KEYS];
    const int b = blockIdx.x, t = threadIdx.x, lane = lane_id(), w = t / WAVE;
    const int s = start ? start[b] : key_start(key, M, shift, b);
    const int rows = (start ? start[b + 1] : key_start(key, M, shift, b + 1)) - s;
    const int k0 = b << shift, keys = min(1 << shift, n - k0);
    for (int c = t; c < NW << shift; c += INC_BLOCK) cnt[c >> shift][c & ((1 << shift) - 1)] = 0;
    __syncthreads();
    const int part = ((rows + NW - 1) / NW + WAVE - 1) / WAVE * WAVE;
    const int p0 = min(w * part, rows), p1 = min(p0 + part, rows);
    // lanes of the wave with this lane's ball
    auto peers_of = [&](int k, bool valid) {
        unsigned long long m = __ballot(valid);
        for (int bit = 0; bit < shift; bit++) {
            const unsigned long long x = __ballot((k >> bit) & 1);
            m &= ((k >> bit) & 1) ? x : ~x;
        }
        return m;
    };
    for (int p = p0 + lane; p - lane < p1; p += WAVE)
        if (p < p1) atomicAdd(&cnt[w][(int)key[s + p] - k0], 1);
    __syncthreads();
    {
        int sum = 0, tot;
        if (t < keys)
            for (int v = 0; v < NW; v++) sum += cnt[v][t];
        int run = block_exclusive_scan<INC_BLOCK>(sum, &tot);
        if (t < keys) inc_start[k0 + t] = s + run;
        if (t < keys)
            for (int v = 0; v < NW; v++) {
                const int c = cnt[v][t];
                cnt[v][t] = run;
                run += c;
            }
    }
    if (b == gridDim.x - 1 && t == 0) inc_start[n] = s + rows;
    __syncthreads();
    for (int p = p0 + lane; p - lane < p1; p += WAVE) {
        const bool valid = p < p1;
        const int k = valid ? (int)key[s + p] - k0 : 0;
        const unsigned long long peers = peers_of(k, valid);
        const int rank = __popcll(peers & ((1ull << lane) - 1ull));
        int at = 0;
        if (valid) at = cnt[w][k] + rank;
        __builtin_amdgcn_wave_barrier();  // every lane has read its counter
        if (valid && rank == 0) cnt[w][k] += __popcll(peers);
        if (valid) inc_slot[s + at] = (int)pay[s + p];
    }
}

// Gradient of ball i: the sum of its incidence slots' contributions, by LPB
// lanes each taking every LPB-th slot and then a fixed tree (deterministic; one
// lane alone walks a chain of two dependent loads per slot, some 15 of them:
// 20 us at 4,001 balls against 4, 34 against 24 at 100,000). Past the balls' blocks, one block sums V and
// A (nb parts to va) where asked to.
constexpr int GATHER_LPB = 8;
__global__ void __launch_bounds__(MEASURE_BLOCK) k_measure_gather(const int *__restrict__ vstart,
                                                                   const int *__restrict__ slot,
                                                                   const double4 *__restrict__ contrib, int n,
                                                                   double *__restrict__ dxyz, double *__restrict__ dr,
                                                                   const double *__restrict__ part, int nb,
                                                                   double *__restrict__ va) {
    constexpr int BALLS = MEASURE_BLOCK / GATHER_LPB;
    if ((int)blockIdx.x * BALLS >= n) {
        measure_total(part, nb, va);
        return;
    }
    const int i = blockIdx.x * BALLS + threadIdx.x / GATHER_LPB, l = threadIdx.x % GATHER_LPB;
    const int q0 = i < n ? vstart[i] : 0, q1 = i < n ? vstart[i + 1] : 0;
    double gx = 0, gy = 0, gz = 0, gr = 0;
    for (int q = q0 + l; q < q1; q += 2 * GATHER_LPB) {
        const bool two = q + GATHER_LPB < q1;
        const int s0 = slot[q], s1 = slot[two ? q + GATHER_LPB : q];
        const double4 c = contrib[s0], e = contrib[s1];
        gx += c.x + (two ? e.x : 0.0);
        gy += c.y + (two ? e.y : 0.0);
        gz += c.z + (two ? e.z : 0.0);
        gr += c.w + (two ? e.w : 0.0);
    }
#pragma unroll
    for (int off = 1; off < GATHER_LPB; off <<= 1) {
        gx += __shfl_xor(gx, off, WAVE);
        gy += __shfl_xor(gy, off, WAVE);
        gz += __shfl_xor(gz, off, WAVE);
        gr += __shfl_xor(gr, off, WAVE);
    }
    if (i >= n || l != 0) return;
    dxyz[3LL * i] = gx;
    dxyz[3LL * i + 1] = gy;
    dxyz[3LL * i + 2] = gz;
    dr[i] = gr;
}

}  // namespace acx
