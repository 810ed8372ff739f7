// HIP kernels of the alpha-complex pipeline for gfx950.
//
// Stages (Masood, Ray, Natarajan, Sec. 3.1 Steps 1-5 and Sec. 4.2-4.5):
//   quantise  -> integer milli-angstrom balls, bounding box, validation
//   binning   -> counting sort of the balls by uniform-grid cell (Sec. 4.2)
//   neighbours-> per ball: every ball whose grown ball (radius^2 W + alpha)
//                meets its own (the only possible AC2 violators of any
//                candidate it belongs to), and the upper candidate edges,
//                Sigma_ortho^1 (Sec. 4.3)
// The later stages are in simplices.hpp and emit.hpp.
#pragma once
#include "common.hpp"
#include "predicates.hpp"
#include "radix.hpp"
#include "rules.hpp"

namespace acx {

struct Stats {
    int minx, miny, minz, maxx, maxy, maxz;
    int wmax, flags;  // flags: 1 invalid value, 2 out of range
    int large;        // balls of a weight above what k_quantise was given
};

// Uniform grid (Sec. 4.2). Cells are numbered in row-major order (x fastest;
// the cells of one grid row are then contiguous in the sorted order), or
// along a Morton (Z-order) curve, the space-filling alternative Sec. 4.2
// names: the bits of the three cell coordinates interleaved, over a cube of
// 2^L cells a side. A batch of molecules has one grid per molecule; their
// cells are numbered one after the other in a single table, so no ball ever
// sees another molecule's balls.
// ORDER_STOP: the grid of a molecule a recorded build could not take (ball k
// of the molecule alone in its cell k, no neighbour scan); see plan.hpp.
enum { ORDER_ROW = 0, ORDER_MORTON = 1, ORDER_STOP = 2 };
constexpr int MORTON_MAX_BITS = 10;  // cell coordinates below 1024: 30-bit codes

struct Grid {
    int ox, oy, oz;   // low corner (mA)
    int s;            // cell side (mA)
    int nx, ny, nz;
    int reach;        // cells to scan on each side for neighbours
    long long base;   // first cell of this grid in the shared cell table
    int a0, a1;       // the molecule's balls: [a0, a1) in input and in sorted order
    int order;        // ORDER_ROW or ORDER_MORTON
};

// v (< 2^10) with two zero bits after each of its bits
__device__ __forceinline__ unsigned spread3(unsigned v) {
    v &= 0x3ffu;
    v = (v | (v << 16)) & 0x030000ffu;
    v = (v | (v << 8)) & 0x0300f00fu;
    v = (v | (v << 4)) & 0x030c30c3u;
    v = (v | (v << 2)) & 0x09249249u;
    return v;
}

// Molecule of ball i (input or sorted index): the last grid with a0 <= i.
__device__ __forceinline__ int mol_of(const Grid *__restrict__ grids, int n_mol, int i) {
    int lo = 0, hi = n_mol - 1;
    while (lo < hi) {
        const int mid = (lo + hi + 1) >> 1;
        if (grids[mid].a0 <= i) lo = mid; else hi = mid - 1;
    }
    return lo;
}

// The molecule that holds all of [i0, i1] (the same in every lane), -1 where none
// does: its grid is then one for the wave, read through the scalar cache and
// held in scalar registers.
__device__ __forceinline__ int mol_of_all(const Grid *__restrict__ grids, int n_mol, int i0, int i1) {
    const int m = mol_of(grids, n_mol, __builtin_amdgcn_readfirstlane(i0));
    return __builtin_amdgcn_readfirstlane(i1) < grids[m].a1 ? m : -1;
}

constexpr int BLOCK = 256;
// Most balls of a group: the simplices of consecutive balls (in sorted order)
// are enumerated, pruned and written by one block.
constexpr int GROUP = BLOCK;

// What a build tells the host while it runs: a block of pinned host memory that
// a kernel writes and the host polls (a copy and a wait for the stream cost
// about 15 us each time). seq: the number of the message, written last.
struct Mail {
    Counters c;
    Stats st;
    unsigned seq;
};
__device__ __forceinline__ void mail_post(Mail *mail, unsigned seq) {
    __threadfence_system();
    __hip_atomic_store(&mail->seq, seq, __ATOMIC_RELEASE, __HIP_MEMORY_SCOPE_SYSTEM);
}

// ---------------------------------------------------------------------------
// Quantise: x -> rint(1000 x) (round half to even), W = R^2. Block b handles
// the balls [tiles[b].x, tiles[b].y) (at most QTILE, all of one molecule; of a
// single molecule of n balls the b-th QTILE, tiles = nullptr) and writes their
// bounding box, flags and number of weights above wlarge; k_stats_reduce folds each molecule's tiles (of a
// single tile there is nothing to fold: it is mailed from here). Block 0 also
// clears the counters of the build, whose first kernel this is. Every load of a
// thread is issued before the first conversion.
constexpr int QTILE = 1024;  // balls per block
__global__ void __launch_bounds__(BLOCK) k_quantise(const double *__restrict__ xyz, const double *__restrict__ r,
                                                     const int2 *__restrict__ tiles, int n, int wlarge, int4 *__restrict__ q,
                                                     Stats *__restrict__ part, Counters *cnt, Mail *mail, unsigned seq) {
    static_assert(sizeof(Counters) % sizeof(int) == 0 && sizeof(Counters) / sizeof(int) <= BLOCK, "cleared as ints");
    if (cnt && blockIdx.x == 0 && threadIdx.x < sizeof(Counters) / sizeof(int)) reinterpret_cast<int *>(cnt)[threadIdx.x] = 0;
    constexpr int PT = QTILE / BLOCK;
    int mn[3] = {INT_MAX, INT_MAX, INT_MAX}, mx[3] = {INT_MIN, INT_MIN, INT_MIN}, wmax = 0, flags = 0, large = 0;
    const int2 tile = tiles ? tiles[blockIdx.x]
                            : make_int2((int)blockIdx.x * QTILE, min(((int)blockIdx.x + 1) * QTILE, n));
    double vx[PT][3], vr[PT];
#pragma unroll
    for (int u = 0; u < PT; u++) {
        const int i = tile.x + (int)threadIdx.x + u * BLOCK;
        const long long k = i < tile.y ? i : tile.x;  // past the tile: any ball of it, not used
#pragma unroll
        for (int a = 0; a < 3; a++) vx[u][a] = xyz[3 * k + a];
        vr[u] = r[k];
    }
#pragma unroll
    for (int u = 0; u < PT; u++) {
        const int i = tile.x + (int)threadIdx.x + u * BLOCK;
        if (i >= tile.y) break;
        int c[3];
#pragma unroll
        for (int a = 0; a < 3; a++) {
            const double v = vx[u][a];
            c[a] = 0;
            if (!isfinite(v)) { flags |= 1; continue; }
            const double s = v * 1000.0;
            if (!(fabs(s) < 524288.0)) { flags |= 2; continue; }
            c[a] = (int)rint(s);
            if (c[a] >= 524288 || c[a] <= -524288) flags |= 2;
            mn[a] = min(mn[a], c[a]);
            mx[a] = max(mx[a], c[a]);
        }
        const double rv = vr[u];
        int W = 0;
        if (!isfinite(rv) || !(rv > 0.0)) {
            flags |= 1;
        } else {
            const double rs = rv * 1000.0;
            if (!(rs < 8192.0)) {
                flags |= 2;
            } else {
                const int R = (int)rint(rs);
                if (R < 1) flags |= 1;
                W = R * R;
            }
        }
        wmax = max(wmax, W);
        large += W > wlarge;
        q[i] = make_int4(c[0], c[1], c[2], W);
    }
#pragma unroll
    for (int off = WAVE / 2; off > 0; off >>= 1) {
#pragma unroll
        for (int a = 0; a < 3; a++) {
            mn[a] = min(mn[a], __shfl_xor(mn[a], off, WAVE));
            mx[a] = max(mx[a], __shfl_xor(mx[a], off, WAVE));
        }
        wmax = max(wmax, __shfl_xor(wmax, off, WAVE));
        flags |= __shfl_xor(flags, off, WAVE);
        large += __shfl_xor(large, off, WAVE);
    }
    __shared__ Stats ws[BLOCK / WAVE];
    const int w = threadIdx.x / WAVE;
    if (lane_id() == 0) ws[w] = Stats{mn[0], mn[1], mn[2], mx[0], mx[1], mx[2], wmax, flags, large};
    __syncthreads();
    if (threadIdx.x == 0) {
        Stats b = ws[0];
        for (int k = 1; k < BLOCK / WAVE; k++) {
            const Stats &o = ws[k];
            b.minx = min(b.minx, o.minx); b.miny = min(b.miny, o.miny); b.minz = min(b.minz, o.minz);
            b.maxx = max(b.maxx, o.maxx); b.maxy = max(b.maxy, o.maxy); b.maxz = max(b.maxz, o.maxz);
            b.wmax = max(b.wmax, o.wmax); b.flags |= o.flags; b.large += o.large;
        }
        part[blockIdx.x] = b;
        if (mail) {
            mail->st = b;
            mail_post(mail, seq);
        }
    }
}

// Block m folds the partials of molecule m's tiles [tile_first[m],
// tile_first[m+1]) into st[m] (of a single molecule: the n_tiles, tile_first =
// nullptr), and mails a single molecule's.
__global__ void __launch_bounds__(BLOCK) k_stats_reduce(const Stats *__restrict__ part, const int *__restrict__ tile_first,
                                                         int n_tiles, Stats *st, Mail *mail, unsigned seq) {
    Stats b{INT_MAX, INT_MAX, INT_MAX, INT_MIN, INT_MIN, INT_MIN, 0, 0, 0};
    const int k0 = tile_first ? tile_first[blockIdx.x] : 0, k1 = tile_first ? tile_first[blockIdx.x + 1] : n_tiles;
    for (int k = k0 + threadIdx.x; k < k1; k += BLOCK) {
        const Stats &o = part[k];
        b.minx = min(b.minx, o.minx); b.miny = min(b.miny, o.miny); b.minz = min(b.minz, o.minz);
        b.maxx = max(b.maxx, o.maxx); b.maxy = max(b.maxy, o.maxy); b.maxz = max(b.maxz, o.maxz);
        b.wmax = max(b.wmax, o.wmax); b.flags |= o.flags; b.large += o.large;
    }
#pragma unroll
    for (int off = WAVE / 2; off > 0; off >>= 1) {
        b.minx = min(b.minx, __shfl_xor(b.minx, off, WAVE));
        b.miny = min(b.miny, __shfl_xor(b.miny, off, WAVE));
        b.minz = min(b.minz, __shfl_xor(b.minz, off, WAVE));
        b.maxx = max(b.maxx, __shfl_xor(b.maxx, off, WAVE));
        b.maxy = max(b.maxy, __shfl_xor(b.maxy, off, WAVE));
        b.maxz = max(b.maxz, __shfl_xor(b.maxz, off, WAVE));
        b.wmax = max(b.wmax, __shfl_xor(b.wmax, off, WAVE));
        b.flags |= __shfl_xor(b.flags, off, WAVE);
        b.large += __shfl_xor(b.large, off, WAVE);
    }
    __shared__ Stats ws[BLOCK / WAVE];
    if (lane_id() == 0) ws[threadIdx.x / WAVE] = b;
    __syncthreads();
    if (threadIdx.x == 0) {
        for (int k = 1; k < BLOCK / WAVE; k++) {
            const Stats &o = ws[k];
            b.minx = min(b.minx, o.minx); b.miny = min(b.miny, o.miny); b.minz = min(b.minz, o.minz);
            b.maxx = max(b.maxx, o.maxx); b.maxy = max(b.maxy, o.maxy); b.maxz = max(b.maxz, o.maxz);
            b.wmax = max(b.wmax, o.wmax); b.flags |= o.flags; b.large += o.large;
        }
        st[blockIdx.x] = b;
        if (mail) {
            mail->st = b;
            mail_post(mail, seq);
        }
    }
}

template <class T>
__global__ void __launch_bounds__(BLOCK) k_fill(T *__restrict__ p, T v, long long n) {
    for (long long i = (long long)blockIdx.x * BLOCK + threadIdx.x; i < n; i += (long long)gridDim.x * BLOCK) p[i] = v;
}

// ---------------------------------------------------------------------------
// Binning (Sec. 4.2): the balls sorted by cell (inside a cell in input order)
// and the dense cell table.
__device__ __forceinline__ long long cell_id(const Grid &g, int cx, int cy, int cz) {
    if (g.order == ORDER_MORTON)
        return (long long)(spread3((unsigned)cx) | (spread3((unsigned)cy) << 1) | (spread3((unsigned)cz) << 2));
    return ((long long)cz * g.ny + cy) * g.nx + cx;
}

__device__ __forceinline__ long long cell_of(const Grid &g, int x, int y, int z) {
    return cell_id(g, (x - g.ox) / g.s, (y - g.oy) / g.s, (z - g.oz) / g.s);
}

// Eight-byte form of a sorted ball for the scan: the low 16 bits of its
// coordinates, and rho = sqrt(W + alpha) rounded up (0 where W + alpha < 0: the
// ball meets none).
typedef short short2v __attribute__((ext_vector_type(2)));
__device__ __forceinline__ int scan_rho(const int4 &a, int aq) {
    const int r2 = a.w + aq;  // below 2^26
    return r2 > 0 ? (int)ceilf(sqrtf((float)r2) * (1.0f + 1.0f / (1 << 20))) : 0;
}
__device__ __forceinline__ int2 scan_ball(const int4 &a, int aq) {
    return make_int2((a.x & 0xffff) | (int)((unsigned)a.y << 16), (a.z & 0xffff) | (scan_rho(a, aq) << 16));
}

// grids = nullptr: one molecule, whose grid is g0 (a kernel argument: no upload).
__device__ __forceinline__ unsigned cell_key(const int4 &a, int i, const Grid &g) {
    return (unsigned)(g.base + (g.order == ORDER_STOP ? i - g.a0 : cell_of(g, a.x, a.y, a.z)));
}

// The balls are sorted by cell in two parts: radix passes over the key bits
// above a bucket of 2^shift consecutive cells make the bucket's balls
// contiguous, and k_bin_finish then orders each bucket by cell in LDS, writes
// its part of the cell table, gathers its balls and checks for equal centres.
// So the low bits need no pass, and the table no count, fill and scan over all
// cells (most of them empty).

// Keys of a radix tile's balls, and the tile's histogram of the first digit.
__global__ void __launch_bounds__(RS_BLOCK) k_cell_hist(const int4 *__restrict__ q, int n, const Grid *__restrict__ grids,
                                                         int n_mol, Grid g0, unsigned *__restrict__ key, int shift,
                                                         int *__restrict__ hist, int tiles) {
    __shared__ int h[RS_BINS];
    h[threadIdx.x] = 0;
    __syncthreads();
    const int base = blockIdx.x * RS_TILE;
    int4 a[RS_IPT];
#pragma unroll
    for (int r = 0; r < RS_IPT; r++) {
        const int i = base + r * RS_BLOCK + (int)threadIdx.x;
        a[r] = i < n ? q[i] : make_int4(0, 0, 0, 0);
    }
    const int m = grids ? mol_of_all(grids, n_mol, base, min(base + RS_TILE, n) - 1) : -1;
#pragma unroll
    for (int r = 0; r < RS_IPT; r++) {
        const int i = base + r * RS_BLOCK + (int)threadIdx.x;
        if (i >= n) break;
        const unsigned k = cell_key(a[r], i, !grids ? g0 : grids[m >= 0 ? m : mol_of(grids, n_mol, i)]);
        key[i] = k;
        atomicAdd(&h[(k >> shift) & (RS_BINS - 1)], 1);
    }
    __syncthreads();
    hist[rs_hist_at(threadIdx.x, blockIdx.x, tiles)] = h[threadIdx.x];
}

// One bucket per block: balls [s, e) of the bucket's cells [k0, k0 + cells).
constexpr int BIN_BLOCK = 256;
constexpr int BIN_ROWS = 2048;   // balls of a bucket held in LDS
constexpr int BIN_SHIFT = 12;    // largest bucket: 2^12 cells
constexpr int BIN_CELLS = 1 << BIN_SHIFT;
// Balls of a cell up to which its balls are compared with each other: both for
// their order and for equal centres. A bucket with a fuller cell, or with more
// than BIN_ROWS balls, goes in chunks with a counter per cell, and looks for equal
// centres among balls of equal hashes (of centre and cell: the bucket's cells may
// be several molecules').
constexpr int BIN_CROWD = 256;

// Hash of a centre (coordinates below 2^20) and its cell: Fibonacci hashing of the
// centre's 63 bits, turned by the cell's.
__device__ __forceinline__ int centre_hash(const int4 &a, unsigned cell) {
    const unsigned long long k = ((unsigned long long)(a.x & 0x1fffff) << 42) | ((unsigned long long)(a.y & 0x1fffff) << 21) |
                                 (unsigned long long)(a.z & 0x1fffff);
    return (int)((k * 0x9E3779B97F4A7C15ull) >> (64 - BIN_SHIFT)) ^ (int)((cell * 0x9E3779B9u) >> (32 - BIN_SHIFT));
}

// Exclusive scan of cnt[0..m) in place (m <= BIN_CELLS, all threads).
__device__ __forceinline__ void bin_scan(int *cnt, int m) {
    constexpr int PT = BIN_CELLS / BIN_BLOCK;
    const int per = (m + BIN_BLOCK - 1) / BIN_BLOCK;  // <= PT
    const int c0 = threadIdx.x * per;
    int s = 0;
    for (int u = 0; u < PT && u < per; u++) s += c0 + u < m ? cnt[c0 + u] : 0;
    int tot;
    int run = block_exclusive_scan<BIN_BLOCK>(s, &tot);
    for (int u = 0; u < PT && u < per; u++)
        if (c0 + u < m) {
            const int c = cnt[c0 + u];
            cnt[c0 + u] = run;
            run += c;
        }
    __syncthreads();
}

// start: first ball of every bucket (nb + 1 entries), or nullptr (searched for). Inside a cell the balls
// keep input order (the radix passes are stable; the LDS places of a cell are
// ranked). gidx, gcell: n entries of scratch each, for a crowded bucket (BIN_CROWD). A build of
// 16,000 balls in one cell 3.9 ms, 146 when the block compared all with each other;
// of 100,000 49 ms, 5,550.
__global__ void __launch_bounds__(BIN_BLOCK) k_bin_finish(const unsigned *__restrict__ key, const unsigned *__restrict__ idx,
                                                           const int *__restrict__ start, int n, int shift, long long ncell,
                                                           const int4 *__restrict__ q, unsigned *__restrict__ gidx,
                                                           unsigned *__restrict__ gcell,
                                                           int *__restrict__ cell_start, int4 *__restrict__ atom,
                                                           int2 *__restrict__ sball, int aq, int *__restrict__ perm,
                                                           Counters *cnt) {
    __shared__ int cc[BIN_CELLS];              // balls per cell, then each cell's first ball, then its end
    __shared__ unsigned short sc[BIN_ROWS];    // cell of each ball, in load order
    __shared__ unsigned short so[BIN_ROWS];    // load positions by cell
    const int b = blockIdx.x, t = threadIdx.x;
    const int s = start ? start[b] : key_start(key, n, shift, b);
    const int rows = (start ? start[b + 1] : key_start(key, n, shift, b + 1)) - s;
    const long long k0 = (long long)b << shift;
    const int cells = (int)min((long long)1 << shift, ncell - k0);
    if (rows == 0) {
        for (int c = t; c < cells; c += BIN_BLOCK) cell_start[k0 + c] = s;
        if (b == gridDim.x - 1 && t == 0) cell_start[ncell] = s;
        return;
    }
    for (int c = t; c < cells; c += BIN_BLOCK) cc[c] = 0;
    __syncthreads();
    bool lds = rows <= BIN_ROWS;
    for (int p = t; p < rows; p += BIN_BLOCK) {
        const int c = (int)((long long)key[s + p] - k0);
        if (lds) sc[p] = (unsigned short)c;
        atomicAdd(&cc[c], 1);
    }
    __syncthreads();
    if (lds && rows > BIN_CROWD) {
        int most = 0;
        for (int c = t; c < cells; c += BIN_BLOCK) most = max(most, cc[c]);
        lds = !__syncthreads_or(most > BIN_CROWD);
    }
    bin_scan(cc, cells);
    for (int c = t; c < cells; c += BIN_BLOCK) cell_start[k0 + c] = s + cc[c];
    if (b == gridDim.x - 1 && t == 0) cell_start[ncell] = s + rows;
    __syncthreads();
    if (lds) {
        for (int p = t; p < rows; p += BIN_BLOCK) so[atomicAdd(&cc[sc[p]], 1)] = (unsigned short)p;
        __syncthreads();
        // cc[c]: end of cell c
        for (int x = t; x < rows; x += BIN_BLOCK) {
            const int p = so[x], c = sc[p];
            const int c0 = c > 0 ? cc[c - 1] : 0, c1 = cc[c];
            int rank = 0;
            for (int y = c0; y < c1; y++) rank += so[y] < p;
            const unsigned id = idx[s + p];
            const int4 a = q[id];
            atom[s + c0 + rank] = a;
            sball[s + c0 + rank] = scan_ball(a, aq);
            perm[s + c0 + rank] = (int)id;
            // equal centres share a cell: compare with the cell's earlier balls
            bool dup = false;
            for (int y = c0; y < c1; y++)
                if (so[y] < p) {
                    const int4 o = q[idx[s + so[y]]];
                    dup |= o.x == a.x && o.y == a.y && o.z == a.z;
                }
            if (dup) cnt->dup = 1;
        }
        return;
    }
    // the rows are in input order: chunk by chunk and wave by wave, each takes the
    // next place of its cell
    const int w = t / WAVE, lane = lane_id();
    unsigned nc = t < rows ? key[s + t] : 0u, nid = t < rows ? idx[s + t] : 0u;
    for (int p0 = 0; p0 < rows; p0 += BIN_BLOCK) {
        const bool valid = p0 + t < rows;
        const int c = valid ? (int)((long long)nc - k0) : 0;
        const unsigned id = nid;
        const int4 a = valid ? q[id] : make_int4(0, 0, 0, 0);
        if (p0 + BIN_BLOCK + t < rows) {  // the next chunk's
            nc = key[s + p0 + BIN_BLOCK + t];
            nid = idx[s + p0 + BIN_BLOCK + t];
        }
        // lanes of the wave with this lane's cell
        unsigned long long peers = __ballot(valid);
        for (int bit = 0; bit < shift; bit++) {
            const unsigned long long x = __ballot((c >> bit) & 1);
            peers &= ((c >> bit) & 1) ? x : ~x;
        }
        const int rank = __popcll(peers & ((1ull << lane) - 1ull));
        int at = 0;
        for (int turn = 0; turn < BIN_BLOCK / WAVE; turn++) {
            if (turn == w && valid) at = cc[c] + rank;
            __builtin_amdgcn_wave_barrier();  // every lane has read its counter
            if (turn == w && valid && rank == 0) cc[c] += __popcll(peers);
            __syncthreads();
        }
        if (valid) {
            atom[s + at] = a;
            sball[s + at] = scan_ball(a, aq);
            perm[s + at] = (int)id;
            gcell[s + at] = (unsigned)c;
        }
    }
    // equal centres in a cell: the balls by hash, each compared with those of its own
    for (int c = t; c < BIN_CELLS; c += BIN_BLOCK) cc[c] = 0;
    __threadfence_block();
    __syncthreads();
    for (int p = t; p < rows; p += BIN_BLOCK) atomicAdd(&cc[centre_hash(atom[s + p], gcell[s + p])], 1);
    __syncthreads();
    bin_scan(cc, BIN_CELLS);
    for (int p = t; p < rows; p += BIN_BLOCK) gidx[s + atomicAdd(&cc[centre_hash(atom[s + p], gcell[s + p])], 1)] = (unsigned)p;
    __threadfence_block();
    __syncthreads();
    bool dup = false;
    for (int p = t; p < rows && !dup; p += BIN_BLOCK) {
        const int4 a = atom[s + p];
        const unsigned c = gcell[s + p];
        const int h = centre_hash(a, c);
        for (int y = h > 0 ? cc[h - 1] : 0; y < cc[h] && !dup; y++) {
            const unsigned o = gidx[s + y];
            if ((int)o >= p) continue;
            const int4 v = atom[s + o];
            dup = v.x == a.x && v.y == a.y && v.z == a.z && gcell[s + o] == c;
        }
    }
    if (dup) cnt->dup = 1;
}

// The whole binning of up to SMALL_BALLS balls on up to SMALL_CELLS cells, in
// one block: keys, cell table, sorted balls and the check for equal centres
// (the passes above cost a small build five launches of some microseconds).
constexpr int SMALL_BLOCK = 1024;
constexpr int SMALL_BALLS = 2048;
constexpr int SMALL_CELLS = 12288;
__global__ void __launch_bounds__(SMALL_BLOCK) k_bin_small(const int4 *__restrict__ q, int n, const Grid *__restrict__ grids,
                                                            int n_mol, Grid g0, int ncell, int *__restrict__ cell_start,
                                                            int4 *__restrict__ atom, int2 *__restrict__ sball,
                                                            int aq, int *__restrict__ perm, Counters *cnt) {
    __shared__ int cc[SMALL_CELLS];
    __shared__ unsigned short sc[SMALL_BALLS], so[SMALL_BALLS];
    const int t = threadIdx.x;
    for (int c = t; c < ncell; c += SMALL_BLOCK) cc[c] = 0;
    __syncthreads();
    for (int i = t; i < n; i += SMALL_BLOCK) {
        const unsigned k = cell_key(q[i], i, grids ? grids[mol_of(grids, n_mol, i)] : g0);
        sc[i] = (unsigned short)k;
        atomicAdd(&cc[k], 1);
    }
    __syncthreads();
    constexpr int PT = SMALL_CELLS / SMALL_BLOCK;
    int c[PT], sum = 0, tot;
#pragma unroll
    for (int u = 0; u < PT; u++) {
        c[u] = t * PT + u < ncell ? cc[t * PT + u] : 0;
        sum += c[u];
    }
    int run = block_exclusive_scan<SMALL_BLOCK>(sum, &tot);
#pragma unroll
    for (int u = 0; u < PT; u++)
        if (t * PT + u < ncell) {
            cell_start[t * PT + u] = run;
            cc[t * PT + u] = run;
            run += c[u];
        }
    if (t == 0) cell_start[ncell] = n;
    __syncthreads();
    for (int i = t; i < n; i += SMALL_BLOCK) so[atomicAdd(&cc[sc[i]], 1)] = (unsigned short)i;
    __syncthreads();
    for (int x = t; x < n; x += SMALL_BLOCK) {
        const int i = so[x], k = sc[i];
        const int c0 = k > 0 ? cc[k - 1] : 0, c1 = cc[k];
        const int4 a = q[i];
        int rank = 0;
        bool dup = false;
        for (int y = c0; y < c1; y++) {
            const int o = so[y];
            if (o >= i) continue;
            rank++;
            const int4 v = q[o];
            dup |= v.x == a.x && v.y == a.y && v.z == a.z;
        }
        atom[c0 + rank] = a;
        sball[c0 + rank] = scan_ball(a, aq);
        perm[c0 + rank] = i;
        if (dup) cnt->dup = 1;
    }
}

// ---------------------------------------------------------------------------
// Neighbour lists and candidate edges (Sec. 4.3, first step). The cells of one
// grid row are contiguous in the sorted order, so a ball scans one contiguous
// range per (dz, dy) row of the cells within `reach`. The pass also decides
// AC2 for the ball as a vertex (Step 5): every ball that could be strictly
// closer in power to its centre is in its neighbour list.
// A candidate edge belongs to its end with the smaller input id: a ball's
// upper row holds the other ends with larger input ids, so that every simplex
// belongs to the ball that comes first in its output row.
//
// The scan tests |p_j - p_i|^2 <= (rho_i + rho_j)^2 on the balls' eight-byte forms
// in 16-bit integers: no coordinate difference in the scanned cells reaches 2^15
// (else, in grids of very large cells, the balls themselves are scanned), so the
// differences are exact, and rho is rounded up, so no neighbour is missed. The
// balls that pass are listed and then tested exactly, where the wave's lanes are
// mostly busy. Seven instructions a scanned ball and eight bytes: with float4
// balls (and addresses, list and row bounds in 64 bits) the kernel was held up
// by the vector caches, 0.9 lines a clock and CU; it is now bound by instruction
// issue (0.8). 283 -> 226 us at 3M atoms and alpha = 0, 23.7 -> 18.4 at 100,000,
// 634 -> 534 for 512 molecules of 5.5M atoms in all.

// Whether the grown balls of two balls meet (d <= rho_a + rho_b) and whether
// their spheres cross (|rho_a - rho_b| <= d too: AC3 of the edge), exactly, for
// balls that passed the scan (so d2 = |b - a|^2 < 2^29), W_a + alpha >= 0; not for
// a ball and itself. L^2 <= 4 rho_a^2 rho_b^2 with L = d^2 - rho_a^2 - rho_b^2; balls one inside
// the other have L < 0. (pp.fast: see spheres_cross.)
enum { BALLS_APART = 0, BALLS_NESTED = 1, BALLS_CROSS = 2 };
__device__ __forceinline__ int balls_meet(const int4 &a, const int4 &b, int d2, const PredParams &pp) {
    const int ra = a.w + (int)pp.aq, rb = b.w + (int)pp.aq;
    if (rb < 0) return BALLS_APART;
    const int L = d2 - ra - rb;
    const bool cross = pp.fast ? (double)L * (double)L <= 4.0 * (double)ra * (double)rb : (i64)L * L <= 4 * (i64)ra * rb;
    return cross ? BALLS_CROSS : L < 0 ? BALLS_NESTED : BALLS_APART;
}
__device__ __forceinline__ int dist2(const int4 &a, const int4 &b) {
    const int dx = b.x - a.x, dy = b.y - a.y, dz = b.z - a.z;
    return m24(dx, dx) + m24(dy, dy) + m24(dz, dz);
}

// (x - o) / s for 0 <= x - o < 2^21: float32 quotient, corrected.
__device__ __forceinline__ int cell_coord(int x, int o, int s, float inv) {
    const int t = x - o;
    int c = (int)((float)t * inv);
    const int r = t - c * s;
    c += (r >= s) - (r < 0);
    return c;
}

// Calls f(j) for every sorted ball j (the ball a itself among them) that passes
// the scan, of the rows part, part + parts, ... of a's cell neighbourhood. sball
// has SCAN_PAD entries more than balls.
constexpr int SCAN_GROUP = 4, SCAN_PAD = SCAN_GROUP - 1;
template <class F>
__device__ __forceinline__ void scan_rows(const Grid &g, const int4 &a, const int4 *__restrict__ atom,
                                          const int2 *__restrict__ sball, const int *__restrict__ cell_start,
                                          const PredParams &pp, int part, int parts, F &&f) {
    const float inv = 1.0f / (float)g.s;
    const int cx = cell_coord(a.x, g.ox, g.s, inv), cy = cell_coord(a.y, g.oy, g.s, inv),
              cz = cell_coord(a.z, g.oz, g.s, inv);
    const int x0 = max(cx - g.reach, 0), x1 = min(cx + g.reach, g.nx - 1);
    const int y0 = max(cy - g.reach, 0), y1 = min(cy + g.reach, g.ny - 1);
    const int z0 = max(cz - g.reach, 0), z1 = min(cz + g.reach, g.nz - 1);
    const int ny = y1 - y0 + 1, rows = ny * (z1 - z0 + 1);
    const bool wide = (long long)(g.reach + 1) * g.s > 32767;
    const int rho = scan_rho(a, (int)pp.aq);
    const short2v mxy = {(short)a.x, (short)a.y}, mzr = {(short)a.z, (short)-rho};
    auto scan_range = [&](int s, int e) {
        if (wide) {
            for (int j = s; j < e; j++) {
                const int4 b = atom[j];
                const float dx = (float)(b.x - a.x), dy = (float)(b.y - a.y), dz = (float)(b.z - a.z);
                const float r = (float)(rho + scan_rho(b, (int)pp.aq)) * (1.0f + 1.0f / (1 << 19));
                if (dx * dx + dy * dy + dz * dz <= r * r) f(j);
            }
            return;
        }
        // the group's loads at fixed offsets of one address (past the range
        // they are some other ball's, or padding, and not used)
        for (int j = s; j < e; j += SCAN_GROUP) {
            const int2 *p = sball + j;
            const int left = e - j;
            int2 b[SCAN_GROUP];
#pragma unroll
            for (int u = 0; u < SCAN_GROUP; u++) b[u] = p[u];
#pragma unroll
            for (int u = 0; u < SCAN_GROUP; u++) {
                const short2v dxy = __builtin_bit_cast(short2v, b[u].x) - mxy;
                const short2v dzr = __builtin_bit_cast(short2v, b[u].y) - mzr;  // (dz, rho_j + rho_i)
                const unsigned d2 = (unsigned)__builtin_amdgcn_sdot2(dxy, dxy, (int)dzr.x * (int)dzr.x, false);
                if ((u < left) & (d2 <= (unsigned)((int)dzr.y * (int)dzr.y))) f(j + u);
            }
        }
    };
    if (rows <= 0 || g.reach < 0) return;  // reach < 0: a stopped recorded build's grid
    if (g.order == ORDER_MORTON) {
        for (int r = part; r < rows; r += parts)
            for (int x = x0; x <= x1; x++) {
                const long long c = g.base + cell_id(g, x, y0 + r % ny, z0 + r / ny);
                scan_range(cell_start[c], cell_start[c + 1]);
            }
        return;
    }
    // a row's balls, or none where all its cells lie farther from the ball than
    // rho + s_g. In float32: the cells' corners are exact, R2 is scaled up by
    // more than the sum's rounding. Cells are below 2^31 in all.
    const float R = (float)(rho + (int)pp.sgc), R2 = R * R * (1.0f + 1.0f / (1 << 19));
    const float side = (float)g.s, last = side - 1.0f, oy = (float)g.oy, oz = (float)g.oz;
    const float ay = (float)a.y, az = (float)a.z;
    const int slab = g.ny * g.nx;
    int y = y0 + part, z = z0, zbase = 0;
    float dz2 = 0.0f;
    auto enter = [&]() {
        const float lo = fmaf((float)z, side, oz);
        const float d = fmaxf(fmaxf(lo - az, az - (lo + last)), 0.0f);
        dz2 = d * d;
        zbase = (int)((unsigned)g.base + (unsigned)z * (unsigned)slab);
    };
    auto wrap = [&]() {
        if (y <= y1) return;
        do {
            y -= ny;
            z++;
        } while (y > y1);
        enter();
    };
    auto bounds = [&]() {
        const float lo = fmaf((float)y, side, oy);
        const float d = fmaxf(fmaxf(lo - ay, ay - (lo + last)), 0.0f);
        if (z > z1 || fmaf(d, d, dz2) > R2) return make_int2(0, 0);
        const int *c = cell_start + (zbase + __mul24(y, g.nx));
        return make_int2(c[x0], c[x1 + 1]);
    };
    enter();
    wrap();
    int2 next = bounds();
    while (z <= z1) {
        // the next row's bounds are loaded while this row is scanned
        const int2 now = next;
        y += parts;
        wrap();
        next = bounds();
        scan_range(now.x, now.y);
    }
}

// One pass: LPB lanes per ball, each scanning its share of the rows into an LDS
// list of LSLOT entries (a launch of few balls is a chain of dependent loads,
// which more lanes shorten; a launch of many fills the GPU with one lane per
// ball, 8 waves per SIMD). The lanes' lists are packed, block by block, into a
// slab of BLOCK / LPB balls x SLOT entries, each ball's upper entries first;
// k_nbr_compact puts the upper rows into place once the block totals are
// scanned. Exact counts are kept unless a row outgrows its room; then
// cnt->overflow is set, and the host counts and fills with k_nbr_rows (same
// result).
// Slot sizes: neighbour_slot.
template <int SLOT, int LPB>
constexpr int nb_waves() { return SLOT == NB_SLOT && LPB == 1 ? 8 : 4; }
template <int SLOT, int LPB, bool SINGLE>
__global__ void __launch_bounds__(BLOCK, (nb_waves<SLOT, LPB>()))
k_neighbours(const int4 *__restrict__ atom, const int2 *__restrict__ sball, const int *__restrict__ perm, int n,
             const Grid *__restrict__ grids, int n_mol, Grid g0, const int *__restrict__ cell_start, PredParams pp,
             int *__restrict__ deg_n, int *__restrict__ deg_up, int *__restrict__ nslab, int *__restrict__ block_tot,
             unsigned char *__restrict__ vgab, long long *__restrict__ vert_min, Counters *cnt) {
    constexpr int BALLS = BLOCK / LPB;             // of a block
    constexpr int LSLOT = SLOT > 32 ? 32 : SLOT;  // of a lane (a mask bit per entry)
    // room of a lane's list: its entries, the ball itself, and one for what
    // does not fit
    constexpr int FULL = LSLOT + 1;
    __shared__ int sn[BLOCK * (FULL + 2)];
    const int b = xcd_block();
    const int i = b * BALLS + (int)threadIdx.x / LPB, part = (int)threadIdx.x % LPB;
    const bool valid = i < n;
    const int4 a = valid ? atom[i] : make_int4(0, 0, 0, 0);
    const int me = valid ? perm[i] : 0;
    const bool ball = valid && a.w + (int)pp.aq >= 0;  // |aq| < 2^26 and W < 2^26
    int at = threadIdx.x;  // entry k of a lane's list at k * BLOCK: a wave's lanes hit distinct banks
    unsigned mask = 0;
    bool gab = true;
    auto scan = [&](const Grid &g) {
        if (!ball) return;
        scan_rows(g, a, atom, sball, cell_start, pp, part, LPB, [&](int j) {
            sn[at] = j;
            at = min(at + BLOCK, (int)threadIdx.x + (FULL + 1) * BLOCK);
        });
    };
    if constexpr (SINGLE) {
        scan(grids ? grids[0] : g0);
    } else {
        const int w0 = b * BALLS + (int)threadIdx.x / WAVE * (WAVE / LPB);
        const int m = w0 < n ? mol_of_all(grids, n_mol, w0, min(w0 + WAVE / LPB, n) - 1) : 0;
        if (m >= 0) scan(grids[m]);
        else if (ball) scan(grids[mol_of(grids, n_mol, i)]);
    }
    int *const rn = sn + threadIdx.x;
    const int listed = at / BLOCK;
    const int kn = min(listed, FULL);
    int cn = 0;
    // the exact test, AC2 of the vertex and AC3 of the edge for each listed
    // ball; the list keeps the neighbours
    for (int k = 0; k < kn; k++) {
        const int j = rn[k * BLOCK];
        if (j == i) continue;
        const int4 bb = atom[j];
        const int id = perm[j];
        const int d2 = dist2(a, bb);
        const int meet = balls_meet(a, bb, d2, pp);
        if (meet == BALLS_APART) continue;
        // power of the ball at a's centre (vertex_violation_sign, ties by id)
        const int P = d2 - bb.w + a.w;
        gab &= P > 0 || (P == 0 && id > me);
        mask |= (unsigned)(id > me && meet == BALLS_CROSS) << (cn & 31);
        if (cn < LSLOT) rn[cn * BLOCK] = j;
        cn++;
    }
    const bool lane_full = listed > FULL || cn > LSLOT;
    cn = min(cn, LSLOT);
    if (cn < 32) mask &= (1u << cn) - 1u;
    // places in the slab: the ball's upper entries, then the others, each by lane
    const int cu = __popc(mask);
    int bn = cn, bu = cu, pu = 0, pl = 0;  // of the ball; before this lane: upper, others
#pragma unroll
    for (int off = 1; off < LPB; off <<= 1) {
        const int xn = __shfl_xor(bn, off, WAVE), xu = __shfl_xor(bu, off, WAVE);
        if (part & off) {
            pu += xu;
            pl += xn - xu;
        }
        bn += xn;
        bu += xu;
    }
    bool bg = gab;
#pragma unroll
    for (int off = 1; off < LPB; off <<= 1) bg &= (bool)__shfl_xor((int)bg, off, WAVE);
    const bool head = part == 0;
    int off3[3], tot3[3];
    block_exclusive_scan3<BLOCK>(head ? bn : 0, head ? bu : 0, head ? bu * (bu - 1) / 2 : 0, off3, tot3);  // bu <= LSLOT LPB
    int first = off3[0];  // of the head lane
    if (LPB > 1) first = __shfl(first, lane_id() & ~(LPB - 1), WAVE);
    if (valid && head) {
        vgab[i] = (unsigned char)(ball && bg);
        // start of the least Size of a kept incident edge, by input id (only
        // read for a ball that fails AC2 at its own centre)
        if (!(ball && bg)) {
            vert_min[me] = ORDERED_POS_INF;
            if (ball) cnt->vng = 1;
        }
        deg_n[i] = bn;
        deg_up[i] = bu;
    }
    if (lane_full || bn > SLOT) cnt->overflow = 1;
    if (threadIdx.x == 0) {
        const int stride = (gridDim.x + 3) & ~3;
        block_tot[b] = tot3[0];               // neighbour entries of the block
        block_tot[stride + b] = tot3[1];      // upper entries of the block
        block_tot[2 * stride + b] = tot3[2];  // pairs of upper entries of one ball
    }
    if (tot3[0] > BALLS * SLOT) return;  // some row outgrew its room: overflow is set
    int *dn = nslab + (long long)b * (BALLS * SLOT) + first;
    pl += bu;
    for (int k = 0; k < cn; k++) {
        const int j = rn[k * BLOCK];
        if ((mask >> k) & 1u) dn[pu++] = j;
        else dn[pl++] = j;
    }
}

// The counted rows of inputs that outgrow the slots, a thread per ball: counts,
// and after their scans the rows (CSR; upper entries with their owner, in scan
// order).
template <bool FILL>
__global__ void __launch_bounds__(BLOCK) k_nbr_rows(const int4 *__restrict__ atom, const int2 *__restrict__ sball,
                                                     const int *__restrict__ perm, int n, const Grid *__restrict__ grids,
                                                     int n_mol, Grid g0, const int *__restrict__ cell_start, PredParams pp,
                                                     int *__restrict__ deg_n, int *__restrict__ deg_up,
                                                     unsigned char *__restrict__ vgab, const int *__restrict__ nbr_start,
                                                     const int *__restrict__ up_start, int *__restrict__ nbr,
                                                     int *__restrict__ up, int *__restrict__ edge_i,
                                                     long long *__restrict__ vert_min, Counters *cnt) {
    const int i = xcd_block() * BLOCK + threadIdx.x;
    if (i >= n) return;
    const int4 a = atom[i];
    const int me = perm[i];
    const bool ball = a.w + (int)pp.aq >= 0;
    int cn = 0, cu = 0;
    bool gab = true;
    const int pn = FILL ? nbr_start[i] : 0, pu = FILL ? up_start[i] : 0;
    if (ball) {
        const Grid g = grids ? grids[mol_of(grids, n_mol, i)] : g0;
        scan_rows(g, a, atom, sball, cell_start, pp, 0, 1, [&](int j) {
            if (j == i) return;
            const int4 bb = atom[j];
            const int meet = balls_meet(a, bb, dist2(a, bb), pp);
            if (meet == BALLS_APART) return;
            const bool upper = perm[j] > me && meet == BALLS_CROSS;
            if (FILL) {
                nbr[pn + cn] = j;
                if (upper) {
                    up[pu + cu] = j;
                    edge_i[pu + cu] = i;
                }
            } else if (vertex_violation_sign(a, i, bb, j, perm) < 0) {
                gab = false;
            }
            cn++;
            cu += upper;
        });
    }
    if (FILL) return;
    deg_n[i] = cn;
    deg_up[i] = cu;
    vgab[i] = (unsigned char)(ball && gab);
    if (!(ball && gab)) {
        vert_min[me] = ORDERED_POS_INF;
        if (ball) cnt->vng = 1;
    }
}

// After a one-pass neighbour search: the neighbour rows stay where the pass
// packed them, in the block's slab (nbr_start[i] points there; the rows of a
// ball are read with its count deg_n[i], so they need not be adjacent across
// blocks). The upper rows, whose entries are the dense candidate-edge ids,
// are written into place (uoff: exclusive scan of the blocks' upper totals),
// each row ordered by input id, with the input id and the owner of every
// entry. pair_base[g]: pairs of upper entries before group g (2^gshift balls;
// poff: exclusive scan of the blocks' pair totals). eng (balls owning an edge
// that fails AC2) starts at 0.
// CB balls a block: 64 where there are few (more blocks, one entry a thread).
template <int SLOT, int LPB, int CB>
__global__ void __launch_bounds__(BLOCK) k_nbr_compact(const int *__restrict__ deg_n, const int *__restrict__ deg_up, int n,
                                                        const int *__restrict__ nslab, const int *__restrict__ uoff,
                                                        const int *__restrict__ poff, const int *__restrict__ perm,
                                                        int *__restrict__ nbr_start, int *__restrict__ up_start,
                                                        int *__restrict__ up, int *__restrict__ up_id,
                                                        int *__restrict__ edge_i, int *__restrict__ pair_base,
                                                        int gshift, unsigned char *__restrict__ eng,
                                                        const int *__restrict__ stop) {
    if (stop && *stop) return;  // a recorded build stopped: the upper rows may not fit
    // the block's upper entries are one contiguous range [gu, gu + totu). Each
    // entry is then a thread's: its rank among its row's ids gives its place
    // (a thread that sorted its own row would hold up its wave for the
    // longest one). UP_LDS entries are held in LDS (at 0.05 atoms per A^3 a
    // block has 900 at alpha = 0 and slots of 16, 2,000 at 2 A^2 and slots of
    // 32); a block with more ranks its entries from global memory, a thread
    // per ball.
    constexpr int UP_LDS = CB * SLOT / 2;
    constexpr int BALLS = BLOCK / LPB;  // balls of a slab
    constexpr int SLABS = CB / BALLS;
    static_assert(SLABS >= 1, "a block's balls are whole slabs");
    __shared__ int s_id[UP_LDS];
    __shared__ unsigned short s_pos[UP_LDS];
    __shared__ unsigned char s_own[UP_LDS];
    __shared__ int s_row[CB + 1];
    const int b = blockIdx.x;
    const int i = b * CB + threadIdx.x;
    const bool mine = (int)threadIdx.x < CB && i < n;
    const int cn = mine ? deg_n[i] : 0, cu = mine ? deg_up[i] : 0;
    const int gu = uoff[b * SLABS], gp = poff[b * SLABS];
    int tot3[3], off3[3];
    block_exclusive_scan3<BLOCK>(cn, cu, cu * (cu - 1) / 2, off3, tot3);
    // the ball's row less the slabs' start: its slab, the rows before it there
    int offn = off3[0];
    if (LPB > 1) {
        offn -= __shfl(offn, lane_id() & ~(BALLS - 1), WAVE);
        offn += (int)threadIdx.x / BALLS * (BALLS * SLOT);
    }
    const int offu = off3[1], totu = tot3[1];
    const int base = b * (CB * SLOT);
    const bool lds = totu <= UP_LDS;
    if ((int)threadIdx.x < CB) s_row[threadIdx.x] = offu;
    if (threadIdx.x == 0) s_row[CB] = totu;
    if (mine) {
        if ((i & ((1 << gshift) - 1)) == 0) pair_base[i >> gshift] = gp + off3[2];
        eng[i] = 0;
        nbr_start[i] = base + offn;
        up_start[i] = gu + offu;
        if (i == n - 1) up_start[n] = gu + offu + cu;
        for (int k = 0; k < cu; k++) {
            if (lds) {
                s_pos[offu + k] = (unsigned short)(offn + k);
                s_own[offu + k] = (unsigned char)threadIdx.x;
            } else {
                const int j = nslab[base + offn + k], id = perm[j];
                int rank = 0;
                for (int r = 0; r < cu; r++) rank += perm[nslab[base + offn + r]] < id;
                const int e = gu + offu + rank;
                up[e] = j;
                up_id[e] = id;
                edge_i[e] = i;
            }
        }
    }
    if (!lds) return;
    __syncthreads();
    for (int k = threadIdx.x; k < totu; k += BLOCK) s_id[k] = perm[nslab[base + s_pos[k]]];
    __syncthreads();
    for (int k = threadIdx.x; k < totu; k += BLOCK) {
        const int o = s_own[k], id = s_id[k];
        const int r0 = s_row[o], r1 = s_row[o + 1];
        int rank = 0;
        for (int q = r0; q < r1; q++) rank += s_id[q] < id;
        const int e = gu + r0 + rank;
        up[e] = nslab[base + s_pos[k]];
        up_id[e] = id;
        edge_i[e] = b * CB + o;
    }
}

// After the counted fill: the upper rows ordered by input id (k_up_ids, then
// k_up_rank), and the pairs of upper entries per group.
__global__ void __launch_bounds__(BLOCK) k_up_ids(const int *__restrict__ up, int E, const int *__restrict__ perm,
                                                   int *__restrict__ id) {
    const int e = blockIdx.x * BLOCK + threadIdx.x;
    if (e < E) id[e] = perm[up[e]];
}

__global__ void __launch_bounds__(BLOCK) k_up_rank(const int *__restrict__ up_in, const int *__restrict__ id_in, int E,
                                                    const int *__restrict__ edge_i, const int *__restrict__ up_start,
                                                    int *__restrict__ up, int *__restrict__ up_id) {
    const int e = blockIdx.x * BLOCK + threadIdx.x;
    if (e >= E) return;
    const int i = edge_i[e], id = id_in[e];
    const int r0 = up_start[i], r1 = up_start[i + 1];
    int rank = 0;
    for (int q = r0; q < r1; q++) rank += id_in[q] < id;
    up[r0 + rank] = up_in[e];
    up_id[r0 + rank] = id;
}

// Pairs of upper entries of each group's balls (a wave each), capped at
// INT_MAX (a group past that leaves no room for pair-sized rows anyway), and
// the start of eng.
__global__ void __launch_bounds__(BLOCK) k_group_pairs(const int *__restrict__ deg_up, int n, int gshift, int groups,
                                                        int *__restrict__ pairs, unsigned char *__restrict__ eng) {
    const int g = blockIdx.x * (BLOCK / WAVE) + threadIdx.x / WAVE;
    if (g >= groups) return;
    const int i1 = min((g + 1) << gshift, n);
    long long v = 0;
    for (int i = (g << gshift) + lane_id(); i < i1; i += WAVE) {
        const long long c = deg_up[i];
        v += c * (c - 1) / 2;
        eng[i] = 0;
    }
    for (int off = WAVE / 2; off > 0; off >>= 1) v += __shfl_xor(v, off, WAVE);
    if (lane_id() == 0) pairs[g] = (int)(v < INT_MAX ? v : INT_MAX);
}

// Block totals of the one-pass neighbour search (nb blocks: neighbour
// entries, upper entries, pairs, each array `stride` entries, a multiple of 4):
// exclusive scans of the last two, and the three totals in Counters. One block
// walks them in chunks of 1024 * NBS_IPT; one launch instead of a scan per
// array.
constexpr int NBS_BLOCK = 1024;
constexpr int NBS_IPT = 4;
__global__ void __launch_bounds__(NBS_BLOCK) k_nbr_scan(const int *__restrict__ tot, int nb, int stride,
                                                         int *__restrict__ uoff, int *__restrict__ poff, Counters *cnt, Mail *mail,
                                                         unsigned seq) {
    long long nn = 0, cu = 0, cp = 0;
    for (int c0 = 0; c0 < nb; c0 += NBS_BLOCK * NBS_IPT) {
        const int base = c0 + threadIdx.x * NBS_IPT;
        int a[NBS_IPT], u[NBS_IPT], p[NBS_IPT];
        load_run<NBS_IPT>(tot, base, nb, a);
        load_run<NBS_IPT>(tot + stride, base, nb, u);
        load_run<NBS_IPT>(tot + 2 * stride, base, nb, p);
        int su = 0, sp = 0;
#pragma unroll
        for (int k = 0; k < NBS_IPT; k++) {
            nn += a[k];
            su += u[k];
            sp += p[k];
        }
        int off[3], t[3];
        block_exclusive_scan3<NBS_BLOCK>(0, su, sp, off, t);
        int ru = (int)cu + off[1], rp = (int)cp + off[2];
#pragma unroll
        for (int k = 0; k < NBS_IPT; k++) {
            const int xu = u[k], xp = p[k];
            u[k] = ru;
            p[k] = rp;
            ru += xu;
            rp += xp;
        }
        store_run<NBS_IPT>(uoff, base, nb, u);
        store_run<NBS_IPT>(poff, base, nb, p);
        cu += t[1];
        cp += t[2];
    }
    __shared__ long long ws[NBS_BLOCK / WAVE];
    for (int off = WAVE / 2; off > 0; off >>= 1) nn += __shfl_xor(nn, off, WAVE);
    if (lane_id() == 0) ws[threadIdx.x / WAVE] = nn;
    __syncthreads();
    if (threadIdx.x == 0) {
        long long t = 0;
        for (int k = 0; k < NBS_BLOCK / WAVE; k++) t += ws[k];
        cnt->Nn = t;
        cnt->E = cu;
        cnt->P = cp;
        if (mail) {
            mail->c = *cnt;
            mail_post(mail, seq);
        }
    }
}

// 64-bit sum of n int32 counts: each block writes its partial to
// out[blockIdx.x]; k_fold_i64 then adds the partials in block order.
__global__ void __launch_bounds__(BLOCK) k_sum_i64(const int *__restrict__ x, long long n, long long *__restrict__ out) {
    __shared__ long long ws[BLOCK / WAVE];
    long long v = 0;
    for (long long i = (long long)blockIdx.x * BLOCK + threadIdx.x; i < n; i += (long long)gridDim.x * BLOCK) v += x[i];
    for (int off = WAVE / 2; off > 0; off >>= 1) v += __shfl_down(v, off, WAVE);
    if (lane_id() == 0) ws[threadIdx.x / WAVE] = v;
    __syncthreads();
    if (threadIdx.x == 0) {
        long long t = 0;
        for (int k = 0; k < BLOCK / WAVE; k++) t += ws[k];
        out[blockIdx.x] = t;
    }
}

__global__ void __launch_bounds__(BLOCK) k_fold_i64(const long long *__restrict__ part, int nb, long long *__restrict__ out) {
    __shared__ long long ws[BLOCK / WAVE];
    long long v = 0;
    for (int k = threadIdx.x; k < nb; k += BLOCK) v += part[k];
    for (int off = WAVE / 2; off > 0; off >>= 1) v += __shfl_down(v, off, WAVE);
    if (lane_id() == 0) ws[threadIdx.x / WAVE] = v;
    __syncthreads();
    if (threadIdx.x == 0) {
        long long t = 0;
        for (int k = 0; k < BLOCK / WAVE; k++) t += ws[k];
        *out = t;
    }
}

}  // namespace acx
