// Emit: the kept simplices as rows of input ids, ascending inside a row, rows
// in lexicographic order, each with its Size (Sec. 2.3; the paper outputs
// membership only).
//
// Every simplex belongs to its least input id, and the pruning kernels hold
// each ball's simplices in output order already. So the rows of ball u start
// where the kept rows of the balls before u end: the balls' kept counts, put
// at their input ids by the last pruning kernel, are scanned (k_rec_*), and
// k_rows writes every kept candidate to its ball's start plus its rank among
// the ball's kept ones. No sort; the writes of a ball are contiguous (balls
// are numbered in no spatial order in general, so consecutive balls of a
// block write to different places).
//
// The merge of a partitioned build, whose rows come from several slabs, sorts:
// rows keyed by their least id with the remaining ids and the Size as payload.
// A bucket is 2^shift consecutive ids (at most EK_KEYS; smaller for small
// inputs, so that there are some hundred buckets). A stable LSD radix sort
// over the key bits above the bucket (8-bit passes) makes every bucket's rows
// contiguous; k_key_starts finds where each bucket starts, and k_emit_block
// finishes one bucket per block in LDS: it loads the bucket's rows, counts the
// rows of each id with LDS atomics, scans the counts, orders the rows by id,
// ranks each row in its id's group by the remaining ids and writes it to its
// final place. Every global access is a contiguous range; no global atomics,
// no scattered writes (a bucket with more rows than LDS holds is finished
// through global scratch instead).
#pragma once
#include "common.hpp"
#include "radix.hpp"
#include "simplices.hpp"

namespace acx {

// Sort payload of a row: the ids after the least, then the Size bits (edges,
// triangles) or the candidate index (tetrahedra, whose Size is read at the
// end: they are few).
template <int K> struct EmitPay;
template <> struct EmitPay<2> { typedef uint3 type; };  // v1, Size bits
template <> struct EmitPay<3> { typedef uint4 type; };  // v1, v2, Size bits
template <> struct EmitPay<4> { typedef uint4 type; };  // v1, v2, v3, candidate

__device__ __forceinline__ uint2 bits_of(double x) {
    const unsigned long long b = (unsigned long long)__double_as_longlong(x);
    return make_uint2((unsigned)b, (unsigned)(b >> 32));
}
__device__ __forceinline__ double double_of(unsigned lo, unsigned hi) {
    return __longlong_as_double((long long)(((unsigned long long)hi << 32) | lo));
}

// Key and payload of a row with ascending input ids v[0..K): key = least id,
// payload = the others and `size` (K = 2, 3) or the row's place c (K = 4).
template <int K>
__device__ __forceinline__ void emit_pack(const int (&v)[4], double size, int c, unsigned &key,
                                          typename EmitPay<K>::type &pay) {
    key = (unsigned)v[0];
    if constexpr (K == 2) {
        const uint2 z = bits_of(size);
        pay = make_uint3((unsigned)v[1], z.x, z.y);
    } else if constexpr (K == 3) {
        const uint2 z = bits_of(size);
        pay = make_uint4((unsigned)v[1], (unsigned)v[2], z.x, z.y);
    } else {
        pay = make_uint4((unsigned)v[1], (unsigned)v[2], (unsigned)v[3], (unsigned)c);
    }
}

// Payloads held in registers as uint4 (a 12-byte uint3 in an array of a
// batch ends up in scratch memory; uint4 stays in registers).
__device__ __forceinline__ uint4 widen(const uint3 &q) { return make_uint4(q.x, q.y, q.z, 0u); }
__device__ __forceinline__ uint4 widen(const uint4 &q) { return q; }
template <class P> __device__ __forceinline__ P narrow(const uint4 &q);
template <> __device__ __forceinline__ uint3 narrow<uint3>(const uint4 &q) { return make_uint3(q.x, q.y, q.z); }
template <> __device__ __forceinline__ uint4 narrow<uint4>(const uint4 &q) { return q; }

template <int K>
__device__ __forceinline__ void pay_ids(const uint4 &q, unsigned (&r)[3]) {
    if constexpr (K == 2) { r[0] = q.x; r[1] = 0; r[2] = 0; }
    else if constexpr (K == 3) { r[0] = q.x; r[1] = q.y; r[2] = 0; }
    else { r[0] = q.x; r[1] = q.y; r[2] = q.z; }
}

template <int K>
__device__ __forceinline__ double pay_size(const uint4 &q, const double *__restrict__ size) {
    if constexpr (K == 2) return double_of(q.y, q.z);
    else if constexpr (K == 3) return double_of(q.z, q.w);
    else return size[q.w];
}

constexpr int EK_SHIFT = 9;              // largest bucket: 2^EK_SHIFT ids
constexpr int EK_KEYS = 1 << EK_SHIFT;
constexpr int EK_BLOCK = 256;
// Rows a block orders in LDS, per dimension. The host picks each dimension's
// bucket size so that its expected largest bucket fits (a row is keyed by its
// least id, so the lowest ids of a randomly numbered input key about K times
// the mean number of rows per id).
template <int K> constexpr int ek_rows() { return K == 4 ? 512 : 2048; }
// What a row holds in LDS besides its 16-bit id in the bucket and its place
// in the order. Edges: only the other id (8 bytes a row, about 18 KB a block,
// eight blocks per CU); the Size bits are read again from the bucket's
// payload when the row is written, from cache, as the block has just read
// them. Triangles and tetrahedra: the whole payload (20 bytes a row; a
// triangle block, about 42 KB, leaves room for three per CU): slim triangle
// rows (six blocks per CU) read the payload twice and were no faster.
template <int K> constexpr bool ek_slim() { return K == 2; }

template <int K>
__device__ __forceinline__ void write_row(int *__restrict__ out, long long pos, unsigned k, const unsigned (&r)[3]) {
    if constexpr (K == 2) {
        *reinterpret_cast<int2 *>(out + pos * 2) = make_int2((int)k, (int)r[0]);
    } else if constexpr (K == 4) {
        *reinterpret_cast<int4 *>(out + pos * 4) = make_int4((int)k, (int)r[0], (int)r[1], (int)r[2]);
    } else {
        out[pos * K] = (int)k;
#pragma unroll
        for (int c = 1; c < K; c++) out[pos * K + c] = (int)r[c - 1];
    }
}

__device__ __forceinline__ bool ids_less(const unsigned (&v)[3], const unsigned (&r)[3]) {
    return v[0] != r[0] ? v[0] < r[0] : (v[1] != r[1] ? v[1] < r[1] : v[2] < r[2]);
}

// Block b finishes bucket b (b < nb): its rows [start[b], start[b + 1]) of key /
// pay are written, in order, to out / out_size at the same places (every row
// before the bucket belongs to smaller ids), with their Sizes as they are. Block 0
// writes the row count start[nb] to *m_out. gkey / gpay (m entries) are scratch
// for a bucket with more than ek_rows<K>() rows.
// start = nullptr: one block takes every row unsorted (rows_in, at most
// ek_rows<K>(); ids below EK_KEYS, shift EK_SHIFT). A few hundred balls then need
// no radix sort.
template <int K>
__global__ void __launch_bounds__(EK_BLOCK) k_emit_block(const unsigned *__restrict__ key,
                                                          const typename EmitPay<K>::type *__restrict__ pay,
                                                          const int *__restrict__ start, int shift, int nb,
                                                          unsigned *__restrict__ gkey,
                                                          typename EmitPay<K>::type *__restrict__ gpay,
                                                          const double *__restrict__ size_in,
                                                          int *__restrict__ out, double *__restrict__ out_size,
                                                          int *__restrict__ m_out, int rows_in = 0) {
    constexpr int NI = K - 1;  // ids after the least
    constexpr bool SLIM = ek_slim<K>();
    constexpr int NW = SLIM ? NI : (K == 2 ? 3 : 4);  // payload words held in LDS
    constexpr int ROWS = ek_rows<K>();
    __shared__ unsigned sid[NW][ROWS];      // the bucket's rows' other ids (payloads), in load order
    __shared__ unsigned short skey[ROWS];   // their ids less the bucket's first
    __shared__ unsigned short sord[ROWS];   // load positions in id order
    // rows per id; then each id's first place; after the ordering, where each
    // id's group ends (= the next id's first place)
    __shared__ int cnt[EK_KEYS];
    __shared__ int wsum[EK_BLOCK / WAVE];
    const int b = blockIdx.x, t = threadIdx.x;
    const bool one = start == nullptr;
    if (b == 0 && t == 0) *m_out = one ? rows_in : start[nb];
    const int bs = one ? 0 : start[b], rows = one ? rows_in : start[b + 1] - bs;
    const unsigned k0 = (unsigned)b << shift;  // the bucket's ids: [k0, k0 + 2^shift), 2^shift <= EK_KEYS
    for (int k = t; k < EK_KEYS; k += EK_BLOCK) cnt[k] = 0;
    __syncthreads();
    const bool lds = rows <= ROWS;
    // counts per id (and, in LDS, the rows' ids); four rows per thread loaded
    // together
    for (int p0 = t; p0 < rows; p0 += 4 * EK_BLOCK) {
        unsigned kk[4];
        uint4 q[4];
#pragma unroll
        for (int u = 0; u < 4; u++) {
            const int p = p0 + u * EK_BLOCK;
            kk[u] = p < rows ? key[bs + p] - k0 : 0u;
            q[u] = p < rows && lds ? widen(pay[bs + p]) : make_uint4(0u, 0u, 0u, 0u);
        }
#pragma unroll
        for (int u = 0; u < 4; u++) {
            const int p = p0 + u * EK_BLOCK;
            if (p >= rows) continue;
            atomicAdd(&cnt[kk[u]], 1);
            if (lds) {
                skey[p] = (unsigned short)kk[u];
                sid[0][p] = q[u].x;
                if constexpr (NW >= 2) sid[1][p] = q[u].y;
                if constexpr (NW >= 3) sid[2][p] = q[u].z;
                if constexpr (NW >= 4) sid[3][p] = q[u].w;
            }
        }
    }
    __syncthreads();
    // exclusive scan of the counts (EK_KEYS / EK_BLOCK per thread)
    {
        constexpr int PT = EK_KEYS / EK_BLOCK;
        int c[PT], s = 0;
#pragma unroll
        for (int u = 0; u < PT; u++) {
            c[u] = cnt[t * PT + u];
            s += c[u];
        }
        const int incl = wave_inclusive_scan(s);
        if (lane_id() == WAVE - 1) wsum[t / WAVE] = incl;
        __syncthreads();
        int run = incl - s;
        for (int w = 0; w < t / WAVE; w++) run += wsum[w];
        __syncthreads();
#pragma unroll
        for (int u = 0; u < PT; u++) {
            cnt[t * PT + u] = run;
            run += c[u];
        }
    }
    __syncthreads();
    if (lds) {
        // order the rows by id (within an id in atomics' order), then rank
        // each row in its id's group by the remaining ids
        for (int p = t; p < rows; p += EK_BLOCK) sord[atomicAdd(&cnt[skey[p]], 1)] = (unsigned short)p;
        __syncthreads();
        for (int s = t; s < rows; s += EK_BLOCK) {
            const int p = sord[s];
            uint4 me;  // Size bits or candidate index
            if constexpr (SLIM) {
                me = widen(pay[bs + p]);
            } else {
                me.x = sid[0][p];
                me.y = sid[NW >= 2 ? 1 : 0][p];
                me.z = sid[NW >= 3 ? 2 : 0][p];
                me.w = NW >= 4 ? sid[NW >= 4 ? 3 : 0][p] : 0u;
            }
            const int k = skey[p];
            const int g0 = k > 0 ? cnt[k - 1] : 0, g1 = cnt[k];
            unsigned r[3];
            r[0] = sid[0][p];
            r[1] = NI >= 2 ? sid[NI >= 2 ? 1 : 0][p] : 0u;
            r[2] = NI >= 3 ? sid[NI >= 3 ? 2 : 0][p] : 0u;
            int rank = 0;
            for (int q = g0; q < g1; q++) {
                const int o = sord[q];
                const unsigned v[3] = {sid[0][o], NI >= 2 ? sid[NI >= 2 ? 1 : 0][o] : 0u,
                                       NI >= 3 ? sid[NI >= 3 ? 2 : 0][o] : 0u};
                rank += (q != s) && ids_less(v, r);
            }
            const long long pos = (long long)bs + g0 + rank;
            write_row<K>(out, pos, k0 + k, r);
            out_size[pos] = pay_size<K>(me, size_in);
        }
        return;
    }
    // a bucket beyond LDS: rows placed in their id's group in global scratch
    // (the bucket's own range of gkey / gpay), ranked from there
    for (int p = t; p < rows; p += EK_BLOCK) {
        const unsigned kk = key[bs + p] - k0;
        const int slot = atomicAdd(&cnt[kk], 1);
        gkey[bs + slot] = kk;
        gpay[bs + slot] = pay[bs + p];
    }
    __threadfence_block();
    __syncthreads();
    for (int s = t; s < rows; s += EK_BLOCK) {
        const int k = (int)gkey[bs + s];
        const int g0 = k > 0 ? cnt[k - 1] : 0, g1 = cnt[k];
        const uint4 me = widen(gpay[bs + s]);
        unsigned r[3];
        pay_ids<K>(me, r);
        int rank = 0;
        for (int q = g0; q < g1; q++) {
            unsigned v[3];
            pay_ids<K>(widen(gpay[bs + q]), v);
            rank += (q != s) && ids_less(v, r);
        }
        const long long pos = (long long)bs + g0 + rank;
        write_row<K>(out, pos, k0 + k, r);
        out_size[pos] = pay_size<K>(me, size_in);
    }
}

// ---------------------------------------------------------------------------
// Scan of the balls' output records (input order): rec[u] = kept edges,
// triangles, tetrahedra and vertex state of ball u becomes base[u] = the rows
// of those dimensions before ball u's, with the vertices' in .w; base[n] = the
// totals (also in Counters). Tiles of REC_TILE balls: k_rec_sums adds up each
// tile, k_rec_prefix scans the tiles in one block (and folds the groups'
// candidate totals), k_rec_apply scans inside the tiles and writes the
// vertices, whose rows are then known. Up to REC_TILE balls one block does
// all of it (k_rec_apply with tile_off = nullptr); up to REC_BLOCK tiles there
// is no k_rec_prefix, each block of k_rec_apply adds up the tiles before its own
// (a launch of 5.6 us at 100,000 balls, 11 at 3M).
constexpr int REC_BLOCK = 1024;
constexpr int REC_IPT = 4;  // records of a lane, a wave apart (coalesced 16-byte accesses)
constexpr int REC_TILE = REC_BLOCK * REC_IPT;

__device__ __forceinline__ int4 operator+(int4 a, int4 b) { return make_int4(a.x + b.x, a.y + b.y, a.z + b.z, a.w + b.w); }
__device__ __forceinline__ int4 operator-(int4 a, int4 b) { return make_int4(a.x - b.x, a.y - b.y, a.z - b.z, a.w - b.w); }

// Counts of ball u's record; vert_min: least Size of a kept incident edge of
// a ball that fails AC2 at its own centre.
__device__ __forceinline__ int4 rec_counts(const int4 &r, const long long *__restrict__ vert_min, int u) {
    return make_int4(r.x, r.y, r.z, r.w > 0 || (r.w == VERT_MAYBE && vert_min[u] != ORDERED_POS_INF));
}

__device__ __forceinline__ int4 wave_inclusive_scan4(int4 v) {
    return make_int4(wave_inclusive_scan(v.x), wave_inclusive_scan(v.y), wave_inclusive_scan(v.z),
                     wave_inclusive_scan(v.w));
}
__device__ __forceinline__ int4 last_lane4(int4 v) {
    return make_int4(__shfl(v.x, WAVE - 1, WAVE), __shfl(v.y, WAVE - 1, WAVE), __shfl(v.z, WAVE - 1, WAVE),
                     __shfl(v.w, WAVE - 1, WAVE));
}

// Sum of v over the waves of a block before this one (v: the same in every
// lane of a wave); *total receives the block's sum.
template <int NT>
__device__ __forceinline__ int4 waves_before4(int4 v, int4 *total) {
    __shared__ int4 wsum[NT / WAVE];
    const int w = threadIdx.x / WAVE;
    if (lane_id() == 0) wsum[w] = v;
    __syncthreads();
    int4 off = make_int4(0, 0, 0, 0), tot = off;
#pragma unroll
    for (int k = 0; k < NT / WAVE; k++) {
        if (k < w) off = off + wsum[k];
        tot = tot + wsum[k];
    }
    __syncthreads();
    *total = tot;
    return off;
}

__global__ void __launch_bounds__(REC_BLOCK) k_rec_sums(const int4 *__restrict__ rec,
                                                         const long long *__restrict__ vert_min, int n,
                                                         int4 *__restrict__ tile_sum, const int *__restrict__ stop) {
    if (stop && *stop) return;
    const int u0 = blockIdx.x * REC_TILE;
    int4 s = make_int4(0, 0, 0, 0);
#pragma unroll
    for (int k = 0; k < REC_IPT; k++) {
        const int u = u0 + k * REC_BLOCK + threadIdx.x;
        if (u < n) s = s + rec_counts(rec[u], vert_min, u);
    }
    int4 tot;
    (void)waves_before4<REC_BLOCK>(last_lane4(wave_inclusive_scan4(s)), &tot);
    if (threadIdx.x == 0) tile_sum[blockIdx.x] = tot;
}

// Totals of a finished scan (one thread), and the capacity check of a
// recorded build's outputs (cap: rows of dimensions 1..3).
struct OutCap {
    int E, T, Q;
};
__device__ __forceinline__ void rec_totals(int4 t, Counters *cnt, bool fixed, OutCap cap, int why) {
    cnt->m0 = t.w;
    cnt->m1 = t.x;
    cnt->m2 = t.y;
    cnt->m3 = t.z;
    if (fixed && (t.x > cap.E || t.y > cap.T || t.z > cap.Q || cnt->overflow)) cnt->stop |= why;
}

// Candidate triangles and tetrahedra of all groups (one block).
template <int NT>
__device__ __forceinline__ void fold_candidates(const int *__restrict__ tri_cnt, const int *__restrict__ tet_cand,
                                                int groups, Counters *cnt) {
    __shared__ long long ws[2][NT / WAVE];
    long long a = 0, b = 0;
    for (int k = threadIdx.x; k < groups; k += NT) {
        a += tri_cnt[k];
        b += tet_cand[k];
    }
    for (int o = WAVE / 2; o > 0; o >>= 1) {
        a += __shfl_xor(a, o, WAVE);
        b += __shfl_xor(b, o, WAVE);
    }
    if (lane_id() == 0) {
        ws[0][threadIdx.x / WAVE] = a;
        ws[1][threadIdx.x / WAVE] = b;
    }
    __syncthreads();
    if (threadIdx.x == 0) {
        a = b = 0;
        for (int k = 0; k < NT / WAVE; k++) {
            a += ws[0][k];
            b += ws[1][k];
        }
        cnt->T = a;
        cnt->Q = b;
    }
}

__global__ void __launch_bounds__(1024) k_rec_prefix(int4 *__restrict__ tile_sum, int tiles,
                                                      const int *__restrict__ tri_cnt, const int *__restrict__ tet_cand,
                                                      int groups, Counters *cnt, int fixed, OutCap cap, int why, Mail *mail,
                                                      unsigned seq) {
    if (fixed && cnt->stop) return;
    int4 carry = make_int4(0, 0, 0, 0);
    for (int c0 = 0; c0 < tiles; c0 += 1024) {
        const int k = c0 + threadIdx.x;
        const int4 v = k < tiles ? tile_sum[k] : make_int4(0, 0, 0, 0);
        int4 tot;
        const int4 in = wave_inclusive_scan4(v);
        const int4 ex = carry + waves_before4<1024>(last_lane4(in), &tot) + (in - v);
        if (k < tiles) tile_sum[k] = ex;
        carry = carry + tot;
    }
    fold_candidates<1024>(tri_cnt, tet_cand, groups, cnt);
    if (threadIdx.x == 0) {
        rec_totals(carry, cnt, fixed, cap, why);
        if (mail) {
            mail->c = *cnt;
            mail_post(mail, seq);
        }
    }
}

// tile_off: the tiles' scanned offsets, or (sums) their sums, which each block
// then adds up itself.
__global__ void __launch_bounds__(REC_BLOCK) k_rec_apply(int4 *__restrict__ rec, const long long *__restrict__ vert_min,
                                                          int n, const int4 *__restrict__ tile_off, int sums,
                                                          int *__restrict__ out,
                                                          double *__restrict__ out_size,
                                                          const int *__restrict__ tri_cnt,
                                                          const int *__restrict__ tet_cand, int groups, Counters *cnt,
                                                          int fixed, OutCap cap, int why, Mail *mail, unsigned seq) {
    if (fixed) {
        // read once for the block: the last block may set it (rec_totals) meanwhile
        __shared__ int stopped;
        if (threadIdx.x == 0) stopped = cnt->stop;
        __syncthreads();
        if (stopped) return;
    }
    // a wave takes REC_IPT runs of WAVE consecutive records
    const int u0 = blockIdx.x * REC_TILE + (threadIdx.x / WAVE) * (WAVE * REC_IPT) + lane_id();
    int4 r[REC_IPT], c[REC_IPT], ex[REC_IPT], s = make_int4(0, 0, 0, 0);
#pragma unroll
    for (int k = 0; k < REC_IPT; k++) r[k] = u0 + k * WAVE < n ? rec[u0 + k * WAVE] : make_int4(0, 0, 0, 0);
#pragma unroll
    for (int k = 0; k < REC_IPT; k++) {
        c[k] = u0 + k * WAVE < n ? rec_counts(r[k], vert_min, u0 + k * WAVE) : r[k];
        const int4 in = wave_inclusive_scan4(c[k]);
        ex[k] = s + (in - c[k]);
        s = s + last_lane4(in);
    }
    int4 tot;
    int4 before = waves_before4<REC_BLOCK>(s, &tot);
    if (sums) {  // at most REC_BLOCK tiles
        const int4 v = (int)threadIdx.x < (int)blockIdx.x ? tile_off[threadIdx.x] : make_int4(0, 0, 0, 0);
        int4 off;
        (void)waves_before4<REC_BLOCK>(last_lane4(wave_inclusive_scan4(v)), &off);
        before = before + off;
        tot = tot + off;  // of the last block: of all
    } else if (tile_off) {
        before = before + tile_off[blockIdx.x];
    }
#pragma unroll
    for (int k = 0; k < REC_IPT; k++) {
        const int u = u0 + k * WAVE;
        if (u >= n) break;
        const int4 at = before + ex[k];
        rec[u] = at;
        if (c[k].w) {
            const double sz = r[k].w > 0 ? -(double)r[k].w : double_from_ordered(vert_min[u]);
            out[at.w] = u;
            out_size[at.w] = sz / 1.0e6;  // mA^2 -> A^2
        }
        if (u == n - 1) rec[n] = at + c[k];
    }
    if (blockIdx.x == gridDim.x - 1 && (sums || !tile_off)) {
        fold_candidates<REC_BLOCK>(tri_cnt, tet_cand, groups, cnt);
        if (threadIdx.x == 0) {
            rec_totals(tot, cnt, fixed, cap, why);
            if (mail) {
                mail->c = *cnt;
                mail_post(mail, seq);
            }
        }
    }
}

// The rows and Sizes of a finished recorded build in one launch (array
// blockIdx.y = 2 d: rows of dimension d, 2 d + 1: their Sizes; all 16-byte
// aligned): a copy call each would cost a launch each. The row counts are the
// build's own, so the host need not know them; a stopped build has no rows.
struct CopyList {
    const int *src[8];
    int *dst[8];
};
__global__ void __launch_bounds__(256) k_copy_list(CopyList l, const Counters *__restrict__ cnt) {
    const int a = blockIdx.y, d = a / 2;
    const int m = cnt->stop ? 0 : d == 0 ? cnt->m0 : d == 1 ? cnt->m1 : d == 2 ? cnt->m2 : cnt->m3;
    const long long n = (long long)m * (a & 1 ? 2 : d + 1), n4 = n / 4;
    const int4 *s4 = reinterpret_cast<const int4 *>(l.src[a]);
    int4 *d4 = reinterpret_cast<int4 *>(l.dst[a]);
    const long long t = (long long)blockIdx.x * 256 + threadIdx.x, stride = (long long)gridDim.x * 256;
    for (long long k = t; k < n4; k += stride) d4[k] = s4[k];
    if (t < n - 4 * n4) l.dst[a][4 * n4 + t] = l.src[a][4 * n4 + t];
}

// Rows of each molecule of a batch: molecule m's d-simplices are rows
// [rows[d][m], rows[d][m + 1]), rows[d] = out + d (n_mol + 1), from the scanned
// records at the molecules' first balls (bound, n_mol + 1 entries).
__global__ void __launch_bounds__(256) k_mol_rows(const int4 *__restrict__ base, const long long *__restrict__ bound,
                                                   int n_mol, long long *__restrict__ out,
                                                   const int *__restrict__ stop) {
    const int m = blockIdx.x * 256 + threadIdx.x;
    if (m > n_mol || (stop && *stop)) return;
    const int4 b = base[bound[m]];
    out[m] = b.w;
    out[(n_mol + 1) + m] = b.x;
    out[2LL * (n_mol + 1) + m] = b.y;
    out[3LL * (n_mol + 1) + m] = b.z;
}

// Kept edges, triangles and tetrahedra of a group to their output rows: ball
// u's first row (base[u]) plus the rank among the ball's kept ones. Waves take
// runs of 64 candidates, each for itself: the kept ones of the lane's ball
// before the lane are counted in the wave's ballot, those of the run's first
// ball before the run by a look back at their status (a block scan per round
// would make every wave wait for the slowest of four scattered writes).
// Bound by scattered requests to memory: balls are numbered in no spatial
// order, so each ball's rows are segments of 15 to 45 bytes of their own (13M
// write and 9M read requests at 3M atoms, 436 us, 50 requests a nanosecond); edges in a
// launch apart from the rest, so that a launch's outputs fit the memory-side
// cache, took 450 in all.
// Kept candidates [first, x) of the ball that owns candidate x = c0 + lane
// (first: the ball's first candidate), given the kept ballot of the run.
__device__ __forceinline__ int rank_in_ball(unsigned long long kept, int lane, int first, int c0, int carry) {
    const unsigned long long before = kept & ((1ull << lane) - 1ull);
    return first > c0 ? __popcll(before >> (first - c0)) : carry + __popcll(before);
}

// Rows of two and four ids as one store each. The arrays may be the caller's, so
// no more than an int's alignment is taken for granted (one 8- or 16-byte store
// all the same: the hardware asks for no more).
typedef int row2 __attribute__((ext_vector_type(2), aligned(4)));
typedef int row4 __attribute__((ext_vector_type(4), aligned(4)));

// A tetrahedron's rank follows from the balls' kept counts (a walk back over its
// ball's tetrahedra took 2.5 ms at a ball with 5,900 of them; 0.08 as this).
// LIST: the kept triangles come from k_tri_final's list.
template <bool LIST>
__global__ void __launch_bounds__(BLOCK) k_rows(Cands cd, PredParams pp, const int4 *__restrict__ base,
                                                 const unsigned char *__restrict__ egab,
                                                 const long long *__restrict__ edge_min,
                                                 const unsigned char *__restrict__ tgab,
                                                 const double *__restrict__ tsize,
                                                 const long long *__restrict__ tri_min,
                                                 Tets tt, const int2 *__restrict__ ball_cnt,
                                                 const int *__restrict__ list, const int *__restrict__ list_cnt,
                                                 int *__restrict__ out1, double *__restrict__ size1,
                                                 int *__restrict__ out2, double *__restrict__ size2,
                                                 int *__restrict__ out3, double *__restrict__ size3,
                                                 const int *__restrict__ stop) {
    if (stop && *stop) return;
    const int g = xcd_block();
    const int b0 = g << cd.gshift, b1 = min(b0 + (1 << cd.gshift), cd.n);
    const int w = threadIdx.x / WAVE, lane = lane_id();
    const int e0 = cd.up_start[b0], e1 = cd.up_start[b1];
    // the balls' input ids and first rows, gathered once (a ball's record lies
    // in a line of its own: read per row they would cost more than the rows)
    __shared__ int ids[GROUP], row0[3][GROUP], lfirst[LIST ? GROUP : 1], qfirst[GROUP];
    {  // first list entry and first tetrahedron of each ball
        int off[3], tot[3];
        const int2 c = b0 + (int)threadIdx.x < b1 ? ball_cnt[b0 + threadIdx.x] : make_int2(0, 0);
        block_exclusive_scan3<BLOCK>(LIST ? c.x : 0, c.y, 0, off, tot);
        if (LIST) lfirst[threadIdx.x] = off[0];
        qfirst[threadIdx.x] = off[1];
    }
    if (b0 + (int)threadIdx.x < b1) {
        const int u = cd.perm[b0 + threadIdx.x];
        const int4 r = base[u];
        ids[threadIdx.x] = u;
        row0[0][threadIdx.x] = r.x;
        row0[1][threadIdx.x] = r.y;
        row0[2][threadIdx.x] = r.z;
    }
    __syncthreads();
    for (int c0 = e0 + w * WAVE; c0 < e1; c0 += BLOCK) {
        const int e = c0 + lane;
        const int st = e < e1 ? egab[e] : FACE_OUT;
        const int i = e < e1 ? cd.edge_i[e] : 0;
        const int first = e < e1 ? cd.up_start[i] : 0;
        const unsigned long long kept = __ballot(st != FACE_OUT);
        const int f0 = __shfl(first, 0, WAVE);
        int carry = 0;
        for (int x = f0; x < c0; x += WAVE) carry += __popcll(__ballot(x + lane < c0 && egab[x + lane] != FACE_OUT));
        if (st == FACE_OUT) continue;
        const int u = ids[i - b0];
        const long long p = row0[0][i - b0] + rank_in_ball(kept, lane, first, c0, carry);
        const double sz = st == FACE_GABRIEL ? edge_size_canon(cd.atom[i], cd.atom[cd.up[e]]) : double_from_ordered(edge_min[e]);
        reinterpret_cast<row2 *>(out1)[p] = row2{u, cd.up_id[e]};
        size1[p] = sz / 1.0e6;  // mA^2 -> A^2
    }
    // a kept triangle to its row
    auto write = [&](int t, int e, int i, int st, int rank) {
        const int u = ids[i - b0];
        const long long p = row0[1][i - b0] + rank;
        const double sz = st == FACE_GABRIEL ? tsize[t] : double_from_ordered(tri_min[t]);
        out2[3 * p] = u;
        out2[3 * p + 1] = cd.up_id[e];
        out2[3 * p + 2] = cd.up_id[cd.tri_f[t]];
        size2[p] = sz / 1.0e6;
    };
    const int t0 = cd.tri_base[g], t1 = t0 + (LIST ? 0 : cd.tri_cnt[g]);
    if (LIST) {
        const int m = list_cnt[g];
        for (int x = threadIdx.x; x < m; x += BLOCK) {
            const int t = list[t0 + x];
            const int e = cd.tri_e[t];
            const int i = cd.edge_i[e];
            write(t, e, i, tgab[t], x - lfirst[i - b0]);
        }
    }
    for (int c0 = t0 + w * WAVE; c0 < t1; c0 += BLOCK) {
        const int t = c0 + lane;
        const int st = t < t1 ? tgab[t] : FACE_OUT;
        const int e = t < t1 ? cd.tri_e[t] : 0;
        const int i = t < t1 ? cd.edge_i[e] : -1;
        const unsigned long long kept = __ballot(st != FACE_OUT);
        // the lane's ball's first triangle, where it lies in the run: after
        // the last lane at or before this one whose ball differs from its
        // predecessor's
        const int prev = __shfl_up(i, 1, WAVE);
        const unsigned long long starts = __ballot(lane > 0 && i != prev) & (~0ull >> (WAVE - 1 - lane));
        const int first = starts ? c0 + (WAVE - 1 - __clzll((long long)starts)) : c0;
        int carry = 0;
        const int i0 = __shfl(i, 0, WAVE);
        for (int x = c0;;) {  // runs of 64 before this one, while they hold that ball's triangles
            x -= WAVE;
            const int y = x + lane;
            const bool same = y >= t0 && cd.edge_i[cd.tri_e[y]] == i0;
            carry += __popcll(__ballot(same && tgab[y] != FACE_OUT));
            if (x <= t0 || !__shfl((int)same, 0, WAVE)) break;
        }
        if (st != FACE_OUT) write(t, e, i, st, rank_in_ball(kept, lane, first, c0, carry));
    }
    const int qb = tt.base(g), qn = tt.kept[g];
    for (int x = threadIdx.x; x < qn; x += BLOCK) {
        const int t = tt.t[qb + x], f2 = tt.t2[qb + x];
        const int e = cd.tri_e[t], i = cd.edge_i[e];
        // the group's tetrahedra are in order, all kept
        const int u = ids[i - b0];
        const long long p = row0[2][i - b0] + (x - qfirst[i - b0]);
        reinterpret_cast<row4 *>(out3)[p] = row4{u, cd.up_id[e], cd.up_id[cd.tri_f[t]], cd.up_id[f2]};
        size3[p] = tt.size[qb + x] / 1.0e6;
    }
}

}  // namespace acx
