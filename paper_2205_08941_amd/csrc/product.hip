// Truncated block-sparse products C <- alpha mask_{P_C}(A B) + beta C in FP64.
//
// The products of atom-block matrices cut back to a spatial-cutoff pattern are
// the operations the paper's linear-scaling solver is built from (Background
// and Current Status) and the part it already started to move to GPUs
// (Meeting the Exascale Challenges).
//
// Work decomposition (gfx950, wave64, FP64 vector FMA):
//   * atoms are taken G at a time as a row group; the union of the group's
//     rows of P_C is cut into runs of JT = 64 / b columns.  A tile is (row
//     group, run); one wavefront owns one tile;
//   * lane l holds column c = l % b of the output blocks (i_a, j), j = run[l / b],
//     for all G rows i_a of the group: G x b FP64 accumulators per lane;
//   * the plan lists, per tile, every k for which some (i_a, k, j) triple
//     exists, with the slots of A_{i_a k} and B_kj.  The wave walks that list:
//     it loads the b x b block A_{i_a k} at a wave-uniform address through the
//     scalar cache (an SGPR operand broadcast to all lanes), each lane loads its
//     column of B_kj once and uses it for all G rows.  Exec masks drop lanes
//     whose (k, j) or (i_a, j) is absent, so only existing triples are summed,
//     in ascending k (deterministic);
//   * the next list entry and its B columns are loaded while the current one
//     is multiplied; tiles are mapped so that each XCD owns a contiguous range
//     of row groups (neighbouring rows share A and B blocks in its L2).
// No zero fill enters the flop count: 2 b^3 per triple (i, k, j) present.
#include "bsm_internal.h"
#include "product_any_b.h"
#include "tiles.h"

#include <algorithm>
#include <climits>
#include <utility>
#include <vector>

namespace bsm {
namespace {

constexpr int kXcd = 8;       // MI355X: 8 XCDs, workgroups dealt round-robin
constexpr int kWaves = 4;     // wavefronts (tiles) per workgroup
constexpr int kMaxRows = 16;  // rows of a tile, at most
// entries past a plan's last that the kernels' prefetch reads: the rings read the slots of entry
// 2 D - 2 past the tile's last and up to 16 slots more than one entry's
constexpr int kSpareEntries = 12;
static_assert(kSpareEntries >= 2 * kMaxRingDepth + 3, "spare entries");
constexpr int kPlanThreads = 256;   // threads of a planner workgroup

__device__ inline int64_t logical_workgroup(int64_t nwg_padded)
{
    const int64_t w = blockIdx.x;
    const int64_t per = nwg_padded / kXcd;
    return (w % kXcd) * per + w / kXcd;
}

// Tile header, ints: rows[G] (atom ids, -1 = padding), cslot[G][JT] (slot of
// (i_a, j) in C or -1).  Entries of tile t: ebeg[t] .. ebeg[t+1], each G + JT
// ints: aslot[G] (slot of (i_a, k) in A or -1), bslot[JT] (slot of (k, j) in B or -1).
template <int B, int G, class T>
__global__ __launch_bounds__(256) void k_product_sgpr(
    int64_t ntiles, int64_t nwg_padded, const int *__restrict__ order, const int *__restrict__ hdr,
    const int64_t *__restrict__ ebeg, const int *__restrict__ ent, const T *__restrict__ vA,
    const T *__restrict__ vB, double *__restrict__ vC, double alpha, double beta)
{
    const int64_t slot = logical_workgroup(nwg_padded) * kWaves + (threadIdx.x >> 6);
    if (slot >= ntiles) return;
    tile_sgpr<B, G, T>(order[slot], hdr, ebeg, ent, vA, vB, vC, alpha, beta);
}

template <int B, int G>
__global__ __launch_bounds__(256) void k_product_f64_dpp(
    int64_t ntiles, int64_t nwg_padded, const int *__restrict__ order, const int *__restrict__ hdr,
    const int64_t *__restrict__ ebeg, const int *__restrict__ ent, const double *__restrict__ vA,
    const double *__restrict__ vB, const double *__restrict__ zblk, double *__restrict__ vC, double alpha,
    double beta)
{
    const int64_t slot = logical_workgroup(nwg_padded) * kWaves + (threadIdx.x >> 6);
    if (slot >= ntiles) return;
    tile_dpp<B, G>(order[slot], hdr, ebeg, ent, vA, vB, zblk, vC, alpha, beta);
}

// One workgroup tile (16 rows x JT columns) per workgroup.
template <int B>
__global__ __launch_bounds__(256) void k_product_wg(
    int64_t ntiles, int64_t nwg_padded, const int *__restrict__ order, const int *__restrict__ hdr,
    const int64_t *__restrict__ ebeg, const int *__restrict__ ent, const double *__restrict__ vA,
    const double *__restrict__ vB, double *__restrict__ vC, double alpha, double beta)
{
    __shared__ double lds[2 * WgTile<B>::kStage];
    const int64_t t = logical_workgroup(nwg_padded);
    if (t >= ntiles) return;   // uniform over the workgroup
    tile_wg<B>(order[t], hdr, ebeg, ent, vA, vB, vC, alpha, beta, lds);
}

// One wave tile per one-wave workgroup, operands through a per-wave LDS ring
// (CP: kPointerCopies, kPackedCopies; kBufferCopies, kPackedBuffers with resources of a_bytes and b_bytes).
template <int B, int G, int D, class T = double, int CP = kPointerCopies, int W = 1, int TR = 0>
__global__ __launch_bounds__(64 * W) void k_product_ring(
    int64_t ntiles, int64_t nwg_padded, const int *__restrict__ order, const int *__restrict__ hdr,
    const int64_t *__restrict__ ebeg, const int *__restrict__ ent, const T *__restrict__ vA,
    const T *__restrict__ vB, const T *__restrict__ zblk, double *__restrict__ vC, double alpha, double beta,
    unsigned a_bytes, unsigned b_bytes)
{
    constexpr int kRing = D * RingEntry<B, G, T>::kStep;   // per wave
    __shared__ __attribute__((aligned(16))) char ring[W * kRing];
    const int64_t t = logical_workgroup(nwg_padded);
    if (t >= ntiles) return;   // uniform over the workgroup
    const int w = W > 1 ? (int)(threadIdx.x >> 6) : 0;
    tile_ring<B, G, D, T, CP, W, TR>(order[t], hdr, ebeg, ent, vA, vB, zblk, vC, alpha, beta,
                                      (lds_char_t *)ring + w * kRing, a_bytes, b_bytes);
}

// Two products sharing B and the patterns (C = A B, C2 = A2 B) on one plan of G / 2
// rows: one wave tile of G rows per one-wave workgroup, B's copies serving both
// (TR = 1: a transposed plan, the launch passing the shared left operand as B).
template <int B, int G, int D, int CP, int TR = 0>
__global__ __launch_bounds__(64) void k_product_ring_pair(
    int64_t ntiles, int64_t nwg_padded, const int *__restrict__ order, const int *__restrict__ hdr,
    const int64_t *__restrict__ ebeg, const int *__restrict__ ent, const double *__restrict__ vA,
    const double *__restrict__ vA2, const double *__restrict__ vB, const double *__restrict__ zblk,
    double *__restrict__ vC, double *__restrict__ vC2, double alpha, double beta, unsigned a_bytes,
    unsigned a2_bytes, unsigned b_bytes)
{
    __shared__ __attribute__((aligned(16))) char ring[D * RingEntry<B, G, double>::kStep];
    const int64_t t = logical_workgroup(nwg_padded);
    if (t >= ntiles) return;
    tile_ring<B, G, D, double, CP, 1, TR, 2>(order[t], hdr, ebeg, ent, vA, vB, zblk, vC, alpha, beta,
                                             (lds_char_t *)ring, a_bytes, b_bytes, vA2, vC2, a2_bytes);
}

// FP64 matrix-core tiles (b = 9, G-row wave tiles, variant 6), one per one-wave workgroup.
template <int G, bool BUF>
__global__ __launch_bounds__(64) void k_product_mfma_f64(
    int64_t ntiles, int64_t nwg_padded, const int *__restrict__ order, const int *__restrict__ hdr,
    const int64_t *__restrict__ ebeg, const int *__restrict__ ent, const double *__restrict__ vA,
    const double *__restrict__ vB, const double *__restrict__ zblk, double *__restrict__ vC, double alpha,
    double beta, unsigned a_bytes, unsigned b_bytes)
{
    __shared__ __attribute__((aligned(16))) char ring[2 * RingEntry<9, G, double>::kBytes];
    const int64_t t = logical_workgroup(nwg_padded);
    if (t >= ntiles) return;
    tile_mfma_f64<G, BUF>(order[t], hdr, ebeg, ent, vA, vB, zblk, vC, alpha, beta, (lds_char_t *)ring, a_bytes,
                          b_bytes);
}

// ---------------------------------------------------------------- operand rounding
// FP64 -> FP32 (round to nearest even); for BF16, the FP32 value rounded again
// to 8 significant bits (nearest even, Inf kept, NaN kept quiet), stored as FP32.
__device__ inline float round_bf16(float x)
{
    unsigned u = __float_as_uint(x);
    if ((u & 0x7f800000u) == 0x7f800000u) {
        if (u & 0x007fffffu) u |= 0x00400000u;
        u &= 0xffff0000u;
    } else {
        u += 0x7fffu + ((u >> 16) & 1u);
        u &= 0xffff0000u;
    }
    return __uint_as_float(u);
}

__global__ void k_round_copy(int64_t n, const double *__restrict__ x, float *__restrict__ y, int bf16)
{
    const int64_t e = (int64_t)blockIdx.x * blockDim.x + threadIdx.x;
    if (e >= n) return;
    const float f = (float)x[e];
    y[e] = bf16 ? round_bf16(f) : f;
}

// 9 x 9 FP64 blocks -> packed BF16 blocks of the matrix-core tiles: row p holds
// elements (p, m), m = 0..8, then 7 zeros (transpose: row p holds (m, p)).
// Rounding as k_round_copy: to FP32, then to BF16, both to nearest even.  blockIdx.y = 0: A
// to pa, 1: B, transposed, to pb.  A workgroup's blocks are read and written in whole lines,
// turned in LDS; with a thread per packed element the reads skipped 7 lanes of 16 and the two
// launches took 2 x 83 us for 512 atoms, 16 A; one launch takes 102 (0.47 GB, 4.6 TB/s).
constexpr int kPackThreads = 256, kPackBlocks = 32;

__global__ __launch_bounds__(kPackThreads) void k_pack_bf16_blocks(int64_t nblk, const double *__restrict__ A,
                                                                   const double *__restrict__ Bm,
                                                                   unsigned short *__restrict__ pa,
                                                                   unsigned short *__restrict__ pb)
{
    constexpr int kVec = 8, kVecs = kPackedBlock / kVec, kLoads = (kPackBlocks * 81 + kPackThreads - 1) / kPackThreads;
    __shared__ unsigned short v[kPackBlocks * 81];
    const int transpose = blockIdx.y;
    const double *__restrict__ x = transpose ? Bm : A;
    unsigned short *__restrict__ y = transpose ? pb : pa;
    const int64_t blk0 = (int64_t)blockIdx.x * kPackBlocks;
    const int nb = (int)min((int64_t)kPackBlocks, nblk - blk0), n = nb * 81;
    x += blk0 * 81;
    double xv[kLoads];
#pragma unroll
    for (int u = 0; u < kLoads; ++u) {
        const int e = threadIdx.x + u * kPackThreads;
        xv[u] = e < n ? x[e] : 0.0;
    }
#pragma unroll
    for (int u = 0; u < kLoads; ++u) {
        const int e = threadIdx.x + u * kPackThreads;
        if (e < n) v[e] = (unsigned short)(__float_as_uint(round_bf16((float)xv[u])) >> 16);
    }
    __syncthreads();
    uint4 *o = reinterpret_cast<uint4 *>(y + blk0 * kPackedBlock);   // context scratch: aligned
    for (int c = threadIdx.x; c < nb * kVecs; c += kPackThreads) {
        const int blk = c / kVecs, q = c - blk * kVecs, p = q >> 1, m0 = 8 * (q & 1);   // half of row p
        unsigned short h[kVec];
#pragma unroll
        for (int i = 0; i < kVec; ++i) {
            const int m = m0 + i;
            h[i] = m < 9 ? v[blk * 81 + (transpose ? m * 9 + p : p * 9 + m)] : (unsigned short)0;
        }
        o[c] = make_uint4(h[0] | (unsigned)h[1] << 16, h[2] | (unsigned)h[3] << 16, h[4] | (unsigned)h[5] << 16,
                          h[6] | (unsigned)h[7] << 16);
    }
}

// BF16 matrix-core product tiles (b = 9, G-row wave tiles), one per one-wave workgroup
// (BUF: packed operands copied through buffer resources of a_bytes and b_bytes).
template <int G, bool BUF>
__global__ __launch_bounds__(64) void k_product_mfma_bf16(
    int64_t ntiles, int64_t nwg_padded, const int *__restrict__ order, const int *__restrict__ hdr,
    const int64_t *__restrict__ ebeg, const int *__restrict__ ent, const unsigned short *__restrict__ pA,
    const unsigned short *__restrict__ pBt, const unsigned short *__restrict__ pz, double *__restrict__ vC,
    double alpha, double beta, unsigned a_bytes, unsigned b_bytes)
{
    __shared__ __attribute__((aligned(16))) char ring[4 * (G + 7) * kPackedBytes];
    const int64_t t = logical_workgroup(nwg_padded);
    if (t >= ntiles) return;
    tile_mfma_bf16<G, BUF>(order[t], hdr, ebeg, ent, pA, pBt, pz, vC, alpha, beta, (lds_char_t *)ring, a_bytes,
                           b_bytes);
}

// ---------------------------------------------------------------- planner
// One workgroup per row group (tile headers) or per tile (entries), all over
// windows of atoms held as bit masks in LDS.  Bound by the reads of the pattern
// rows it merges (from L2: a group's tiles share them) and, per entry written,
// 4 (G + JT) bytes.  A thread per group or tile that merged its rows one column
// at a time (the former planner) spent its time in dependent loads on a nearly
// empty chip: the 16 A x 16 A -> 16 A plan of 4096 atoms took 137 ms, one of the
// 216-atom frames 5 ms.
// The section compiles as plain C++ too, where a workgroup is one thread: the
// planner's checks on the CPU run it that way.
#if defined(__HIPCC__)
#define BSM_PLAN_SHARED __shared__
// a launch's workgroups in rows of gridDim.x (its threads along x must stay below 2^32)
__device__ inline int64_t plan_item() { return (int64_t)blockIdx.y * gridDim.x + blockIdx.x; }
__device__ inline void plan_sync() { __syncthreads(); }
__device__ inline int plan_place(int64_t item);   // where an item's totals go
__device__ inline void plan_or(unsigned *p, unsigned v) { atomicOr(p, v); }
__device__ inline void plan_or(unsigned long long *p, unsigned long long v) { atomicOr(p, v); }
__device__ inline void plan_min(int *p, int v) { atomicMin(p, v); }
// exclusive sum over the workgroup's threads, and the total; every thread calls it
__device__ inline unsigned plan_scan(unsigned v, unsigned &total)
{
    __shared__ unsigned part[kPlanThreads / 64];
    const int lane = threadIdx.x & 63, w = threadIdx.x >> 6;
    unsigned x = v;
    for (int off = 1; off < 64; off <<= 1) {
        const unsigned y = __shfl_up(x, off, 64);
        if (lane >= off) x += y;
    }
    if (lane == 63) part[w] = x;
    __syncthreads();
    unsigned base = 0, tot = 0;
    for (int q = 0; q < kPlanThreads / 64; ++q) {
        if (q < w) base += part[q];
        tot += part[q];
    }
    __syncthreads();
    total = tot;
    return base + x - v;
}
#else
#define BSM_PLAN_SHARED static
#define __launch_bounds__(n)
constexpr int kPlanThreads = 1;
inline int64_t plan_item() { return blockIdx.x; }
inline void plan_sync() {}
inline int plan_place(int64_t) { return 0; }
inline void plan_or(unsigned *p, unsigned v) { *p |= v; }
inline void plan_or(unsigned long long *p, unsigned long long v) { *p |= v; }
inline void plan_min(int *p, int v) { *p = min(*p, v); }
inline unsigned plan_scan(unsigned v, unsigned &total)
{
    total = v;
    return 0;
}
#endif

// Tiles add their triples and rows to one of kTotalLanes places, a cache line each: one place for all
// took the atomics of thousands of tiles in turn (k_tile_entries<0>, 216 atoms, b = 9: 70 -> 15 us).
constexpr int kTotalLanes = 64, kTotalStride = 16;
constexpr int kUnionWords = 4096;   // bit words of a column window (131072 atoms)
constexpr int kEntryWindow = 1024;  // atoms k of an entry window

// Columns of the group's rows of P_C (slots lo..hi) inside the window that starts
// at k0, as bits in `bits`; the words used are cleared first.
__device__ inline void union_bits(unsigned *bits, int words, int k0, int lo, int hi, const int *__restrict__ cC)
{
    const int t = threadIdx.x, nt = blockDim.x;
    for (int w = t; w < words; w += nt) bits[w] = 0u;
    plan_sync();
    for (int p = lo + t; p < hi; p += nt) {
        const int d = cC[p] - k0;
        if (d >= 0 && d < 32 * words) plan_or(&bits[d >> 5], 1u << (d & 31));
    }
    plan_sync();
}

// First and last column of a group's rows of P_C (no row is empty: its diagonal is there).
// Windows span these only: over all atoms, each of a long system's groups would clear and scan
// words for every atom of it.
__device__ inline void group_reach(const int *__restrict__ rpC, const int *__restrict__ cC, int i0, int gr, int &first,
                                   int &last)
{
    first = 0x7fffffff;
    last = 0;
    for (int a = 0; a < gr; ++a) {
        first = min(first, cC[rpC[i0 + a]]);
        last = max(last, cC[rpC[i0 + a + 1] - 1]);
    }
}

// One workgroup per row group: tiles that the union of the group's rows of P_C takes.
__global__ __launch_bounds__(kPlanThreads) void k_group_union(int n, int G, const int *__restrict__ rpC,
                                                              const int *__restrict__ cC, int jt,
                                                              int *__restrict__ ntile)
{
    BSM_PLAN_SHARED unsigned bits[kUnionWords];
    const int g = blockIdx.x;
    const int i0 = g * G, gr = min(G, n - i0);
    const int lo = rpC[i0], hi = rpC[i0 + gr];   // the group's rows follow each other
    int first, last;
    group_reach(rpC, cC, i0, gr, first, last);
    unsigned cnt = 0;
    for (int64_t k0 = first; k0 <= last; k0 += 32 * kUnionWords) {
        const int words = (int)min((int64_t)kUnionWords, (last - k0) / 32 + 1);
        union_bits(bits, words, (int)k0, lo, hi, cC);
        for (int w = threadIdx.x; w < words; w += blockDim.x) cnt += __popc(bits[w]);
        plan_sync();
    }
    unsigned total;
    plan_scan(cnt, total);
    if (threadIdx.x == 0) ntile[g] = ((int)total + jt - 1) / jt;
}

// One workgroup per row group: write the tile headers of its runs.  The group's
// union of P_C columns is cut into runs of jt columns, in ascending column order
// (order 0) or grouped by the set of the group's rows whose P_C row holds the
// column (order 1: row sets in descending bit order, ascending columns inside a
// set).  With order 1 a tile's columns share their output rows, so a row
// multiplies in a tile only where it has outputs; the two orders give the same
// products.  scr: per plan 5 + G arrays of ntiles * jt ints, each group using its
// tiles' range: union columns, row sets and union positions in ping-pong pairs,
// and the C slots of every (column, row).  Order 1 sorts the union positions by a
// stable radix sort on 4 row-set bits at a time, each thread counting and placing
// a run of consecutive positions.
__global__ __launch_bounds__(kPlanThreads) void k_group_tiles(int n, int G, int jt, int order,
                                                              const int *__restrict__ rpC,
                                                              const int *__restrict__ cC,
                                                              const int64_t *__restrict__ toff, int64_t ntiles,
                                                              int *__restrict__ hdr, int *__restrict__ tcols,
                                                              int *__restrict__ scr)
{
    BSM_PLAN_SHARED unsigned bits[kUnionWords], rank[kUnionWords];
    BSM_PLAN_SHARED unsigned hist[16 * kPlanThreads];
    const int g = blockIdx.x, t = threadIdx.x, nt = blockDim.x;
    const int hs = G + G * jt;
    const int i0 = g * G, gr = min(G, n - i0);
    const int lo = rpC[i0], hi = rpC[i0 + gr];
    const int64_t t0 = toff[g], cap = ntiles * jt, o = t0 * jt;
    const int room = (int)(toff[g + 1] - t0) * jt;   // columns of the group's tiles
    int *col = scr + o, *m0 = scr + cap + o, *m1 = scr + 2 * cap + o, *x0 = scr + 3 * cap + o,
        *x1 = scr + 4 * cap + o, *sl = scr + 5 * cap + o * G;
    for (int64_t e = t; e < (int64_t)room * G; e += nt) sl[e] = -1;
    // the union's columns in ascending order, and every (column, row)'s C slot
    int first, last;
    group_reach(rpC, cC, i0, gr, first, last);
    unsigned cnt = 0;
    for (int64_t kw = first; kw <= last; kw += 32 * kUnionWords) {
        const int k0 = (int)kw, words = (int)min((int64_t)kUnionWords, (last - kw) / 32 + 1);
        union_bits(bits, words, k0, lo, hi, cC);
        const int per = (words + nt - 1) / nt, w0 = min(words, t * per), w1 = min(words, w0 + per);
        unsigned mine = 0, total;
        for (int w = w0; w < w1; ++w) mine += __popc(bits[w]);
        unsigned run = cnt + plan_scan(mine, total);
        for (int w = w0; w < w1; ++w) {
            rank[w] = run;
            run += __popc(bits[w]);
        }
        plan_sync();
        for (int p = lo + t; p < hi; p += nt) {
            const int k = cC[p], d = k - k0;
            if (d < 0 || d >= 32 * words) continue;
            int a = 0;
            while (p >= rpC[i0 + a + 1]) ++a;
            const int u = (int)(rank[d >> 5] + __popc(bits[d >> 5] & ((1u << (d & 31)) - 1u)));
            col[u] = k;
            sl[(int64_t)u * G + a] = p;
        }
        cnt += total;
        plan_sync();
    }
    const int nu = (int)cnt;
    if (order == 1) {
        for (int u = t; u < nu; u += nt) {
            int set = 0;
            for (int a = 0; a < gr; ++a) set |= (sl[(int64_t)u * G + a] >= 0 ? 1 : 0) << a;
            m0[u] = set;
            x0[u] = u;
        }
        plan_sync();
        const int seg = (nu + nt - 1) / nt, s0 = min(nu, t * seg), s1 = min(nu, s0 + seg);
        for (int bit = 0; bit < gr; bit += 4) {
            for (int v = 0; v < 16; ++v) hist[v * nt + t] = 0u;
            for (int x = s0; x < s1; ++x) hist[(15 - ((m0[x] >> bit) & 15)) * nt + t] += 1u;
            plan_sync();
            // positions: digit by digit (present rows first), thread by thread
            unsigned mine = 0, total;
            for (int v = 0; v < 16; ++v) mine += hist[16 * t + v];
            unsigned run = plan_scan(mine, total);
            for (int v = 0; v < 16; ++v) {
                const unsigned h = hist[16 * t + v];
                hist[16 * t + v] = run;
                run += h;
            }
            plan_sync();
            for (int x = s0; x < s1; ++x) {
                const int m = m0[x];
                const unsigned w = hist[(15 - ((m >> bit) & 15)) * nt + t]++;
                m1[w] = m;
                x1[w] = x0[x];
            }
            plan_sync();
            int *tm = m0, *tx = x0;
            m0 = m1;
            x0 = x1;
            m1 = tm;
            x1 = tx;
        }
    }
    for (int x = t; x < room; x += nt) {
        const int64_t tile = t0 + x / jt;
        const int q = x % jt;
        int *h = hdr + tile * hs;
        if (q == 0)
            for (int a = 0; a < G; ++a) h[a] = (a < gr) ? i0 + a : -1;
        const int u = x < nu ? (order == 1 ? x0[x] : x) : -1;
        tcols[tile * jt + q] = u >= 0 ? col[u] : -1;
        for (int a = 0; a < G; ++a) h[G + a * jt + q] = u >= 0 ? sl[(int64_t)u * G + a] : -1;
    }
}

// One workgroup per (tile, chunk of k in [c n / nch, (c + 1) n / nch)): the k for
// which some (i_a, k, j) triple exists, in ascending order.  MODE 0 counts
// entries and triples per (tile, chunk), MODE 1 writes the entries; a tile's
// chunks follow each other, so its entries stay in ascending k.  The tile's last
// chunk writes the padding entry that makes the tile's count even (its count
// includes it, k_pad_counts).  Each window of kEntryWindow atoms is held as two
// masks per k, the rows a with (i_a, k) in P_A and the columns x with (k, j_x) in
// P_B, filled from the tile's G + jt pattern rows, 64 threads to a row.  A window
// starts at the first k that a row still reaches, and the last is the last that
// both A rows and B columns reach: over all windows of a long system, a tile that
// reaches a few of them spent its time in empty ones (plan and product, 327680
// atoms, b = 2, 4 A: 337 -> 9.5 ms; 110592 atoms, b = 4, 6 A: 89 -> 9.8 ms; 16 A of
// 4096 atoms, whose tiles reach every window, 11.18 and 11.32).  An A row
// (B column) of an entry with no live triple would only meet zero blocks or
// outputs outside P_C: it is dropped, so that the kernels neither copy nor
// multiply it.  W = 2 (tiles shared by two waves): each entry is two halves, one
// per wave and its jt / 2 columns, each with the A slots of the rows that have a
// live triple in those columns and then those columns' B slots.
template <int MODE>
__global__ __launch_bounds__(kPlanThreads) void k_tile_entries(
    int64_t ntiles, int nch, int natoms, int G, int jt, int W, int tr, const int *__restrict__ hdr,
    const int *__restrict__ tcols, const int *__restrict__ rpA, const int *__restrict__ cA,
    const int *__restrict__ tmA, const int *__restrict__ rpB, const int *__restrict__ cB,
    const int *__restrict__ tmB, int64_t *__restrict__ nent, unsigned long long *__restrict__ triples,
    unsigned long long *__restrict__ rowwork, const int64_t *__restrict__ ebeg, int *__restrict__ ent)
{
    constexpr int kRows = kMaxRows + 64;
    BSM_PLAN_SHARED unsigned am[kEntryWindow];             // rows present; then rows live (per half)
    BSM_PLAN_SHARED unsigned long long bm[kEntryWindow];   // columns present; then columns live
    BSM_PLAN_SHARED int eidx[MODE == 1 ? kEntryWindow : 1];
    BSM_PLAN_SHARED int beg[kRows], end[kRows], nxt[kRows];
    BSM_PLAN_SHARED unsigned long long cmask[kMaxRows];    // columns with an output in row a
    BSM_PLAN_SHARED int reach[2][2];                       // first k of the A rows, of the B columns: now, next
    const int64_t tc = plan_item();
    if (tc >= ntiles * nch) return;
    const int64_t t = tc / nch;
    const int c = (int)(tc - t * nch);
    const int k0 = (int)((int64_t)c * natoms / nch), k1 = (int)((int64_t)(c + 1) * natoms / nch);
    const int hs = G + G * jt, es = W * G + jt, jh = jt / W, nr = G + jt;
    const int *h = hdr + t * hs;
    const bool one = k1 - k0 <= kEntryWindow;   // one window: nothing to skip
    const int tid = threadIdx.x, nt = blockDim.x;
    const int sub = nt >= 64 ? 64 : nt, lane = tid % sub, grp = tid / sub, ngrp = nt / sub;
    for (int r = tid; r < nr; r += nt) {
        const int i = r < G ? h[r] : tcols[t * jt + (r - G)];
        const int *cols = r < G ? cA : cB, *rp = r < G ? rpA : rpB;
        int lo = i >= 0 ? rp[i] : 0;
        const int e = i >= 0 ? rp[i + 1] : 0;
        if (k0 > 0) {   // first position at or past k0
            int hi = e;
            while (lo < hi) {
                const int mid = (lo + hi) >> 1;
                if (cols[mid] < k0) lo = mid + 1;
                else hi = mid;
            }
        }
        beg[r] = lo;
        end[r] = e;
    }
    if (tid == 0) reach[0][0] = reach[0][1] = one ? k0 : k1;
    for (int a = tid; a < G; a += nt) {
        unsigned long long m = 0;
        for (int x = 0; x < jt; ++x)
            if (h[G + a * jt + x] >= 0) m |= 1ull << x;
        cmask[a] = m;
    }
    plan_sync();
    const unsigned long long half0 = W == 1 ? ~0ull : (1ull << jh) - 1ull;
    int64_t w = (MODE == 1) ? ebeg[tc] : 0;
    unsigned cnt = 0, tri = 0, rw = 0;
    if (!one) {
        for (int r = tid; r < nr; r += nt)
            if (beg[r] < end[r]) plan_min(&reach[0][r < G ? 0 : 1], (r < G ? cA : cB)[beg[r]]);
        plan_sync();
    }
    for (int now = 0;; now ^= 1) {
        const int ka = reach[now][0], kb = reach[now][1], kw = min(ka, kb);
        if (max(ka, kb) >= k1) break;   // no k left that both reach
        const int ke = k1 - kw > kEntryWindow ? kw + kEntryWindow : k1, len = ke - kw;
        for (int d = tid; d < len; d += nt) {
            am[d] = 0u;
            bm[d] = 0ull;
        }
        if (tid == 0) reach[now ^ 1][0] = reach[now ^ 1][1] = k1;
        plan_sync();
        for (int r = grp; r < nr; r += ngrp) {
            const int *cols = r < G ? cA : cB;
            const int b0 = beg[r], b1 = end[r];
            for (int p = b0 + lane; p <= b1; p += sub) {
                const int k = p < b1 ? cols[p] : 0x7fffffff;
                if (k >= ke) {   // the first position past the window starts the next one
                    if (p == b0 || cols[p - 1] < ke) {
                        nxt[r] = p;
                        if (k < k1) plan_min(&reach[now ^ 1][r < G ? 0 : 1], k);
                    }
                    break;
                }
                if (r < G) plan_or(&am[k - kw], 1u << r);
                else plan_or(&bm[k - kw], 1ull << (r - G));
            }
        }
        plan_sync();
        // each thread takes a run of consecutive k
        const int per = (len + nt - 1) / nt, d0 = min(len, tid * per), d1 = min(len, d0 + per);
        unsigned mine = 0;
        for (int d = d0; d < d1; ++d) {
            const unsigned ra = am[d];
            const unsigned long long cb = bm[d];
            unsigned live = 0;   // rows live in the first half, from bit 16 in the second
            unsigned long long cl = 0;
            if (ra != 0u && cb != 0ull)
                for (int a = 0; a < G; ++a) {
                    if (!((ra >> a) & 1u)) continue;
                    const unsigned long long m = cmask[a] & cb;
                    if (m == 0ull) continue;
                    cl |= m;
                    if (m & half0) live |= 1u << a;
                    if (m & ~half0) live |= 0x10000u << a;
                    if (MODE == 0) tri += (unsigned)(__popc((unsigned)m) + __popc((unsigned)(m >> 32)));
                }
            mine += cl != 0ull ? 1u : 0u;
            if (MODE == 0) rw += (unsigned)__popc(live);   // rows multiplied
            if (MODE == 1) {
                am[d] = live;
                bm[d] = cl;
            }
        }
        if (MODE == 0) {
            cnt += mine;
        } else {
            unsigned total;
            unsigned e = plan_scan(mine, total);
            for (int d = d0; d < d1; ++d) eidx[d] = bm[d] != 0ull ? (int)e++ : -1;
            int *ew = ent + w * es;
            for (int64_t x = tid; x < (int64_t)total * es; x += nt) ew[x] = -1;
            plan_sync();
            for (int r = grp; r < nr; r += ngrp) {
                const int *cols = r < G ? cA : cB, *tm = r < G ? tmA : tmB;
                const int b0 = beg[r], b1 = nxt[r];
                for (int p = b0 + lane; p < b1; p += sub) {
                    const int d = cols[p] - kw, q = eidx[d];
                    if (q < 0) continue;
                    int *eq = ew + (int64_t)q * es;
                    if (r < G) {
                        const unsigned live = am[d] >> r;
                        const int s = tr ? tm[p] : p;   // slot of (i, k); tr: of (k, i)
                        if (live & 1u) eq[r] = s;
                        if (live & 0x10000u) eq[G + jh + r] = s;
                    } else {
                        const int x = r - G, hf = x / jh;
                        if ((bm[d] >> x) & 1ull) eq[hf * (G + jh) + G + x - hf * jh] = tr ? p : tm[p];   // (k, j); tr: (j, k)
                    }
                }
            }
            w += total;
        }
        plan_sync();
        for (int r = tid; r < nr; r += nt) beg[r] = nxt[r];
        plan_sync();
    }
    if (MODE == 1) {
        if (c == nch - 1 && w < ebeg[tc + 1])   // the padding entry: multiplies nothing
            for (int x = tid; x < es; x += nt) ent[w * es + x] = -1;
    } else {
        unsigned scnt, stri, srw;
        plan_scan(cnt, scnt);
        plan_scan(tri, stri);
        plan_scan(rw, srw);
        if (tid == 0) {
            nent[tc] = scnt;
            atomicAdd(triples + plan_place(tc), (unsigned long long)stri);   // integers: order-independent
            atomicAdd(rowwork + plan_place(tc), (unsigned long long)srw);
        }
    }
}

// One thread per tile: make the tile's entry count even by counting a padding
// entry in its last chunk.
__global__ void k_pad_counts(int64_t ntiles, int nch, int64_t *__restrict__ nent)
{
    const int64_t t = (int64_t)blockIdx.x * blockDim.x + threadIdx.x;
    if (t >= ntiles) return;
    int64_t sum = 0;
    for (int c = 0; c < nch; ++c) sum += nent[t * nch + c];
    if (sum & 1) nent[t * nch + nch - 1] += 1;
}

// One thread per tile: the tile's entry range from the (tile, chunk) ranges.
__global__ void k_tile_ebeg(int64_t ntiles, int nch, const int64_t *__restrict__ ebeg_tc, int64_t *__restrict__ ebeg)
{
    const int64_t t = (int64_t)blockIdx.x * blockDim.x + threadIdx.x;
    if (t > ntiles) return;
    ebeg[t] = ebeg_tc[t * nch];
}

// One thread per tile of a transposed plan: C slots of (i, j) -> slots of (j, i).
__global__ void k_map_cslots(int64_t ntiles, int G, int jt, const int *__restrict__ tmC, int *__restrict__ hdr)
{
    const int64_t t = (int64_t)blockIdx.x * blockDim.x + threadIdx.x;
    if (t >= ntiles) return;
    int *h = hdr + t * (G + G * jt) + G;
    for (int x = 0; x < G * jt; ++x)
        if (h[x] >= 0) h[x] = tmC[h[x]];
}

__global__ __launch_bounds__(1024) void k_scan64(int64_t n, const int64_t *__restrict__ in, int64_t *__restrict__ out,
                                                 int64_t *host, const int *__restrict__ in32)
{   // host: also the total, in pinned memory; in32: ints instead of `in`
    __shared__ long long part[1024];
    const int t = threadIdx.x, nt = blockDim.x;
    const int64_t chunk = (n + nt - 1) / nt;
    const int64_t lo = min(n, (int64_t)t * chunk), hi = min(n, lo + chunk);
    long long s = 0;
    for (int64_t k = lo; k < hi; ++k) s += in32 ? in32[k] : in[k];
    part[t] = s;
    __syncthreads();
    for (int off = 1; off < nt; off <<= 1) {
        long long v = (t >= off) ? part[t - off] : 0;
        __syncthreads();
        part[t] += v;
        __syncthreads();
    }
    long long run = part[t] - s;
    for (int64_t k = lo; k < hi; ++k) {
        out[k] = run;
        run += in32 ? in32[k] : in[k];
    }
    if (t == nt - 1) {
        out[n] = part[t];
        if (host) *host = part[t];
    }
}

__device__ inline int plan_place(int64_t item) { return (int)(item & (kTotalLanes - 1)) * kTotalStride; }

// One wave: the sums of the places (triples, then rows multiplied) to pinned memory.
__global__ __launch_bounds__(kTotalLanes) void k_plan_totals(const unsigned long long *__restrict__ totals,
                                                             unsigned long long *host)
{
    unsigned long long v[2] = {totals[threadIdx.x * kTotalStride], totals[threadIdx.x * kTotalStride + 1]};
    for (int off = kTotalLanes / 2; off > 0; off >>= 1)
        for (int k = 0; k < 2; ++k) v[k] += __shfl_xor(v[k], off, kTotalLanes);
    if (threadIdx.x < 2) host[threadIdx.x] = v[threadIdx.x];
}

template <int B, int G, class T = double>
void launch_bg(hipStream_t st, const Plan *plan, const T *A, const T *Bm, double *C, double alpha,
               double beta)
{
    const int64_t nwg = (plan->ntiles + kWaves - 1) / kWaves;
    const int64_t nwg_padded = ((nwg + kXcd - 1) / kXcd) * kXcd;
    k_product_sgpr<B, G, T><<<(unsigned)nwg_padded, 64 * kWaves, 0, st>>>(
        plan->ntiles, nwg_padded, plan->order.as<int>(), plan->hdr.as<int>(), plan->ebeg.as<int64_t>(),
        plan->ent.as<int>(), A, Bm, C, alpha, beta);
}

template <int B, int G>
void launch_dpp(hipStream_t st, const Plan *plan, const double *A, const double *Bm, double *C, double alpha,
                double beta, const double *zblk)
{
    const int64_t nwg = (plan->ntiles + kWaves - 1) / kWaves;
    const int64_t nwg_padded = ((nwg + kXcd - 1) / kXcd) * kXcd;
    k_product_f64_dpp<B, G><<<(unsigned)nwg_padded, 64 * kWaves, 0, st>>>(
        plan->ntiles, nwg_padded, plan->order.as<int>(), plan->hdr.as<int>(), plan->ebeg.as<int64_t>(),
        plan->ent.as<int>(), A, Bm, zblk, C, alpha, beta);
}

template <int B>
void launch_wg(hipStream_t st, const Plan *plan, const double *A, const double *Bm, double *C, double alpha,
               double beta)
{
    const int64_t nwg_padded = ((plan->ntiles + kXcd - 1) / kXcd) * kXcd;
    k_product_wg<B><<<(unsigned)nwg_padded, 256, 0, st>>>(plan->ntiles, nwg_padded, plan->order.as<int>(),
                                                         plan->hdr.as<int>(), plan->ebeg.as<int64_t>(),
                                                         plan->ent.as<int>(), A, Bm, C, alpha, beta);
}

// Ring depth of packed copies.  Paired tiles hold twice the sums to an entry and hide the copies one
// entry ahead; a second one cost them: 512 atoms, b = 4, 16 A, 701 us with two, 851 with three; 1000
// atoms, 14 A, 2429 and 2546 (216 atoms 104 and 107).
constexpr int kPackedDepth = 3, kPackedPairDepth = 2;

template <int B, int G, int D, class T = double, int W = 1, int TR = 0>
void launch_ring_t(hipStream_t st, const Plan *plan, const T *A, const T *Bm, double *C, double alpha, double beta,
                   const T *zblk, int64_t a_bytes, int64_t b_bytes)
{
    const int64_t nwg_padded = ((plan->ntiles + kXcd - 1) / kXcd) * kXcd;
    auto go = [&](auto kern, bool buf) {
        kern<<<(unsigned)nwg_padded, 64 * W, 0, st>>>(
            plan->ntiles, nwg_padded, plan->order.as<int>(), plan->hdr.as<int>(), plan->ebeg.as<int64_t>(),
            plan->ent.as<int>(), A, Bm, zblk, C, alpha, beta, buf ? (unsigned)a_bytes : 0u, buf ? (unsigned)b_bytes : 0u);
    };
    // variants 4 and 5: buffer copies when both operands fit a buffer resource; else 64-bit addresses
    const bool buf = (plan->variant == 4 || plan->variant == 5) && a_bytes <= (int64_t)kBufMaxBytes &&
                     b_bytes <= (int64_t)kBufMaxBytes;
    if constexpr (B == 4) {
        if (can_pack(A, Bm)) {
            if (buf) go(k_product_ring<B, G, kPackedDepth, T, kPackedBuffers, W, TR>, true);
            else go(k_product_ring<B, G, kPackedDepth, T, kPackedCopies, W, TR>, false);
            return;
        }
    }
    // two-row tiles serve products of few tiles, whose waves run alone on their SIMDs: one entry
    // further ahead covers the copies' latency
    constexpr int DD = G == 2 && D == 2 && W == 1 ? 3 : D;
    if (buf) go(k_product_ring<B, G, DD, T, kBufferCopies, W, TR>, true);
    else go(k_product_ring<B, G, DD, T, kPointerCopies, W, TR>, false);
}

// Transposed plans (one-wave tiles of 4 or 8 rows, depth 2) compute C^T = B^T A^T:
// the kernel's A operand is B and its B operand is A.
template <int B, int G, int D, class T = double, int W = 1>
void launch_ring(hipStream_t st, const Plan *plan, const T *A, const T *Bm, double *C, double alpha, double beta,
                 const T *zblk, int64_t a_bytes, int64_t b_bytes)
{
    if constexpr (W == 1 && D == 2) {
        if (plan->transposed) {
            launch_ring_t<B, G, D, T, W, 1>(st, plan, Bm, A, C, alpha, beta, zblk, b_bytes, a_bytes);
            return;
        }
    }
    if (plan->transposed) throw Error{BSM_EINVAL, "transposed plan without a transposed kernel"};
    launch_ring_t<B, G, D, T, W, 0>(st, plan, A, Bm, C, alpha, beta, zblk, a_bytes, b_bytes);
}

template <int G>
void launch_mfma_f64(hipStream_t st, const Plan *plan, const double *A, const double *Bm, double *C, double alpha,
                     double beta, const double *zblk, int64_t a_bytes, int64_t b_bytes)
{
    const int64_t nwg_padded = ((plan->ntiles + kXcd - 1) / kXcd) * kXcd;
    const bool buf = a_bytes <= (int64_t)kBufMaxBytes && b_bytes <= (int64_t)kBufMaxBytes;
    if (buf)
        k_product_mfma_f64<G, true><<<(unsigned)nwg_padded, 64, 0, st>>>(
            plan->ntiles, nwg_padded, plan->order.as<int>(), plan->hdr.as<int>(), plan->ebeg.as<int64_t>(),
            plan->ent.as<int>(), A, Bm, zblk, C, alpha, beta, (unsigned)a_bytes, (unsigned)b_bytes);
    else
        k_product_mfma_f64<G, false><<<(unsigned)nwg_padded, 64, 0, st>>>(
            plan->ntiles, nwg_padded, plan->order.as<int>(), plan->hdr.as<int>(), plan->ebeg.as<int64_t>(),
            plan->ent.as<int>(), A, Bm, zblk, C, alpha, beta, 0u, 0u);
}

template <int B>
void launch_b(hipStream_t st, const Plan *plan, const double *A, const double *Bm, double *C, double alpha,
              double beta, const double *zblk, int64_t a_bytes, int64_t b_bytes)
{
    if constexpr (B == 9) {
        if (plan->variant == 6) {   // FP64 matrix cores, direct one-wave plans of 4 or 8 rows
            if (plan->transposed) throw Error{BSM_EINVAL, "variant 6 takes direct plans"};
            switch (plan->G) {
                case 4: launch_mfma_f64<4>(st, plan, A, Bm, C, alpha, beta, zblk, a_bytes, b_bytes); return;
                case 8: launch_mfma_f64<8>(st, plan, A, Bm, C, alpha, beta, zblk, a_bytes, b_bytes); return;
                default: throw Error{BSM_EINVAL, "variant 6 takes 4 or 8 rows per tile"};
            }
        }
    }
    if constexpr (B >= 5 && B != 9) {
        if (plan->variant == 4) {
            launch_any_b(st, plan, A, Bm, C, alpha, beta, zblk, a_bytes, b_bytes);
            return;
        }
    }
    if constexpr (B == 9 || B == 4) {
        if (plan->variant == 5) {   // LDS rings, tiles shared by two waves
            switch (plan->G) {
                case 4: launch_ring<B, 4, 2, double, 2>(st, plan, A, Bm, C, alpha, beta, zblk, a_bytes, b_bytes); return;
                case 8: launch_ring<B, 8, 2, double, 2>(st, plan, A, Bm, C, alpha, beta, zblk, a_bytes, b_bytes); return;
                default: throw Error{BSM_EINVAL, "variant 5 takes 4 or 8 rows per tile"};
            }
        }
        if (plan->variant == 3 || plan->variant == 4) {   // LDS ring, depth 3 or 2
            const bool deep = plan->variant == 3;
            switch (plan->G) {
                case 2: deep ? launch_ring<B, 2, 3>(st, plan, A, Bm, C, alpha, beta, zblk, a_bytes, b_bytes)
                             : launch_ring<B, 2, 2>(st, plan, A, Bm, C, alpha, beta, zblk, a_bytes, b_bytes); return;
                case 4: deep ? launch_ring<B, 4, 3>(st, plan, A, Bm, C, alpha, beta, zblk, a_bytes, b_bytes)
                             : launch_ring<B, 4, 2>(st, plan, A, Bm, C, alpha, beta, zblk, a_bytes, b_bytes); return;
                case 8: launch_ring<B, 8, 2>(st, plan, A, Bm, C, alpha, beta, zblk, a_bytes, b_bytes); return;
                default: break;
            }
        }
        if (plan->variant == 2) {
            launch_wg<B>(st, plan, A, Bm, C, alpha, beta);
            return;
        }
        if (plan->variant == 1) {
            switch (plan->G) {
                case 2: launch_dpp<B, 2>(st, plan, A, Bm, C, alpha, beta, zblk); return;
                case 4: launch_dpp<B, 4>(st, plan, A, Bm, C, alpha, beta, zblk); return;
                default: break;
            }
        }
    }
    switch (plan->G) {
        case 2: launch_bg<B, 2>(st, plan, A, Bm, C, alpha, beta); break;
        case 4: launch_bg<B, 4>(st, plan, A, Bm, C, alpha, beta); break;
        case 8: launch_bg<B, 8>(st, plan, A, Bm, C, alpha, beta); break;
        default: throw Error{BSM_EINVAL, "rows per wave must be 2, 4 or 8"};
    }
}

template <int B>
void launch_b32(hipStream_t st, const Plan *plan, const float *A, const float *Bm, double *C, double alpha,
                double beta, const float *zblk, int64_t a_bytes, int64_t b_bytes)
{
    if constexpr (B >= 5 && B != 9) {
        if (plan->variant == 4) {
            launch_any_b(st, plan, A, Bm, C, alpha, beta, zblk, a_bytes, b_bytes);
            return;
        }
    }
    if constexpr (B == 9 || B == 4) {
        if (plan->variant == 5) {   // LDS rings, tiles shared by two waves, FP32 operands
            switch (plan->G) {
                case 4: launch_ring<B, 4, 2, float, 2>(st, plan, A, Bm, C, alpha, beta, zblk, a_bytes, b_bytes); return;
                case 8: launch_ring<B, 8, 2, float, 2>(st, plan, A, Bm, C, alpha, beta, zblk, a_bytes, b_bytes); return;
                default: throw Error{BSM_EINVAL, "variant 5 takes 4 or 8 rows per tile"};
            }
        }
        if (plan->variant == 3 || plan->variant == 4) {   // LDS ring, FP32 operands
            switch (plan->G) {
                case 2: launch_ring<B, 2, 2, float>(st, plan, A, Bm, C, alpha, beta, zblk, a_bytes, b_bytes); return;
                case 4: launch_ring<B, 4, 2, float>(st, plan, A, Bm, C, alpha, beta, zblk, a_bytes, b_bytes); return;
                case 8: launch_ring<B, 8, 2, float>(st, plan, A, Bm, C, alpha, beta, zblk, a_bytes, b_bytes); return;
                default: break;
            }
        }
    }
    switch (plan->G) {
        case 2: launch_bg<B, 2, float>(st, plan, A, Bm, C, alpha, beta); break;
        case 4: launch_bg<B, 4, float>(st, plan, A, Bm, C, alpha, beta); break;
        case 8: launch_bg<B, 8, float>(st, plan, A, Bm, C, alpha, beta); break;
        default: throw Error{BSM_EINVAL, "rows per wave must be 2, 4 or 8"};
    }
}

#define BSM_FOR_EACH_B(X) \
    X(1) X(2) X(3) X(4) X(5) X(6) X(7) X(8) X(9) X(10) X(11) X(12) X(13) X(14) X(15) X(16)

}  // namespace

int default_rows_per_wave(int b) { return b >= 5 ? 4 : (b == 4 ? 4 : 2); }
int default_variant(int b) { return (b == 9 || b == 4) ? 4 : 0; }

namespace {
// What the two stages of building a plan share: the tiles of P_C (the same for the
// direct and the transposed plan of a product) and the entry ranges of a counted plan.
struct TileSet {
    int G = 0, waves = 1, jt = 0, ng = 0;
    int64_t nt = 0;
    DevBuf hdr, groups, columns;              // what the pointers below point into
    int *ntile = nullptr, *tcols = nullptr, *scr = nullptr;
    int64_t *toff = nullptr;
};
// Workgroups of a launch over the tiles
dim3 tile_grid(int64_t nt)
{
    const int64_t x = std::min<int64_t>(nt, 1 << 22);
    return dim3((unsigned)x, (unsigned)((nt + x - 1) / x));
}
struct EntryCount {
    DevBuf buf;   // what the pointers below point into
    int64_t *nent = nullptr, *ebeg = nullptr;
    int64_t ne = 0;
    unsigned long long ntri[2] = {0, 0};   // triples, rows multiplied
};

// Launch order: within each span of `span` consecutive row groups, chunk position
// first, so that the groups' tiles over similar columns run together and share B
// blocks in L2.  One workgroup per row group, one thread per tile of it.
__global__ void k_tile_order(int ng, int span, const int *__restrict__ ntile, const int64_t *__restrict__ toff,
                             int *__restrict__ order)
{
    const int g = blockIdx.x, g0 = g - g % span, g1 = min(ng, g0 + span);
    for (int q = threadIdx.x; q < ntile[g]; q += blockDim.x) {
        int64_t pos = toff[g0];
        for (int o = g0; o < g1; ++o) pos += min(ntile[o], q) + ((o < g && ntile[o] > q) ? 1 : 0);
        order[pos] = (int)(toff[g] + q);
    }
}

// Columns of a group, at most, that k_cluster_tiles orders (more keep the order of their row sets).
constexpr int kClusterCols = 2048;
// Weight of a differing row in the distance of two columns, Angstrom^2.
constexpr float kClusterRow = 20.0f;

// One wave per row group: take the group's columns tile by tile, each tile the column
// farthest from the group and the jt - 1 columns nearest to it, by squared distance plus
// kClusterRow per row that holds an output in one of the two only.  A tile's columns then
// need nearly the same k: fewer entries, fewer idle lanes and fewer copied blocks than
// runs of the row-set order, whose columns share rows but lie anywhere on the sphere.
// Counted on 4096 atoms, b = 9: 16 A x 16 A -> 16 A 13% fewer entries and 6% fewer rows
// multiplied, 8 A x 10 A -> 18 A 12% and 12%, 10 A x 6 A -> 16 A 11% and 10%.
// hdr and tcols hold the row-set order (k_group_tiles) and are rewritten; scr as there.
// Ties go to the lower column, so the tiles do not depend on timing.  A serial chain of picks, each a minimum
// over the wave: by DPP moves instead of shuffles 101 -> 78 us for 216 atoms.
__global__ __launch_bounds__(64) void k_cluster_tiles(int n, int G, int jt, const double *__restrict__ pos, double bx,
                                                      double by, double bz, const int64_t *__restrict__ toff,
                                                      int64_t ntiles, int *__restrict__ hdr, int *__restrict__ tcols,
                                                      const int *__restrict__ scr)
{
    __shared__ float px[kClusterCols], py[kClusterCols], pz[kClusterCols];
    __shared__ unsigned key[kClusterCols];
    __shared__ int set[kClusterCols], pick[64];
    const int g = blockIdx.x, lane = threadIdx.x, hs = G + G * jt;
    const int i0 = g * G, gr = min(G, n - i0);
    const int64_t t0 = toff[g], cap = ntiles * jt, o = t0 * jt;
    const int nt = (int)(toff[g + 1] - t0), room = nt * jt;
    const int *col = scr + o, *sl = scr + 5 * cap + o * G;
    if (room > kClusterCols) return;
    const double box[3] = {bx, by, bz};
    double cen[3];
    for (int d = 0; d < 3; ++d) {
        double s = 0.0;
        for (int a = 0; a < gr; ++a) {
            const double v = pos[3 * (i0 + a) + d] - pos[3 * i0 + d];
            s += v - box[d] * rint(v / box[d]);
        }
        cen[d] = pos[3 * i0 + d] + s / gr;
    }
    int left = 0;   // columns not yet taken
    for (int u = lane; u < room; u += 64) {
        int m = 0;
        for (int a = 0; a < G; ++a) m |= (sl[(int64_t)u * G + a] >= 0 ? 1 : 0) << a;
        set[u] = m;   // 0: no column here
        float r[3] = {0.f, 0.f, 0.f};
        if (m != 0)
            for (int d = 0; d < 3; ++d) {
                const double v = pos[3 * col[u] + d] - cen[d];
                r[d] = (float)(v - box[d] * rint(v / box[d]));
            }
        px[u] = r[0];
        py[u] = r[1];
        pz[u] = r[2];
        left += m != 0 ? 1 : 0;
    }
    for (int off = 32; off > 0; off >>= 1) left += __shfl_xor(left, off, 64);
    __syncthreads();
    const float fx = (float)bx, fy = (float)by, fz = (float)bz, ix = 1.f / fx, iy = 1.f / fy, iz = 1.f / fz;
    // A column's key: its distance's upper bits and, below them, the column itself, so that one
    // integer minimum gives the nearest (distances are told apart to 1 part in 4096, then by column).
    auto pack = [](float d, int u) { return (__float_as_uint(d) & ~(unsigned)(kClusterCols - 1)) | (unsigned)u; };
    constexpr unsigned kNone = 0xffffffffu;
    auto least = [&](unsigned v) {   // over the wave: within rows of 16, then across them, to the last lane
        const auto with = [&](auto C, auto R) {
            v = min(v, (unsigned)__builtin_amdgcn_update_dpp((int)kNone, (int)v, decltype(C)::value, decltype(R)::value,
                                                             0xf, false));
        };
        with(std::integral_constant<int, 0x111>{}, std::integral_constant<int, 0xf>{});   // row_shr 1, 2, 4, 8
        with(std::integral_constant<int, 0x112>{}, std::integral_constant<int, 0xf>{});
        with(std::integral_constant<int, 0x114>{}, std::integral_constant<int, 0xf>{});
        with(std::integral_constant<int, 0x118>{}, std::integral_constant<int, 0xf>{});
        with(std::integral_constant<int, 0x142>{}, std::integral_constant<int, 0xa>{});   // row_bcast 15, 31
        with(std::integral_constant<int, 0x143>{}, std::integral_constant<int, 0xc>{});
        return (unsigned)__builtin_amdgcn_readlane((int)v, 63);
    };
    for (int t = 0; t < nt; ++t) {
        unsigned best = kNone;
        for (int u = lane; u < room; u += 64)   // the farthest: the least inverse square
            if (set[u] != 0) best = min(best, pack(1.0f / (1.0f + px[u] * px[u] + py[u] * py[u] + pz[u] * pz[u]), u));
        const int seed = (int)(least(best) & (kClusterCols - 1));
        const float sx = px[seed], sy = py[seed], sz = pz[seed];
        const int ss = set[seed];
        for (int u = lane; u < room; u += 64) {
            const int m = set[u];
            float dx = px[u] - sx, dy = py[u] - sy, dz = pz[u] - sz;
            dx -= fx * rintf(dx * ix);
            dy -= fy * rintf(dy * iy);
            dz -= fz * rintf(dz * iz);
            key[u] = m == 0 ? kNone
                            : pack((dx * dx + dy * dy + dz * dz) + kClusterRow * (float)__popc((unsigned)(m ^ ss)), u);
        }
        const int take = min(jt, left);
        if (lane == 0) {
            key[seed] = kNone;
            set[seed] = 0;
            pick[0] = seed;
        }
        __syncthreads();
        for (int q = 1; q < take; ++q) {
            best = kNone;
            for (int u = lane; u < room; u += 64) best = min(best, key[u]);
            const int u = (int)(least(best) & (kClusterCols - 1));
            if (lane == 0) {
                key[u] = kNone;
                set[u] = 0;
                pick[q] = u;
            }
            __syncthreads();
        }
        left -= take;
        for (int x = lane; x < (G + 1) * jt; x += 64) {
            const int a = x / jt, q = x - a * jt, u = q < take ? pick[q] : -1;
            if (a == G) tcols[(t0 + t) * jt + q] = u >= 0 ? col[u] : -1;
            else hdr[(t0 + t) * hs + G + a * jt + q] = u >= 0 ? sl[(int64_t)u * G + a] : -1;
        }
        __syncthreads();
    }
}

// cluster: tiles of near columns (k_cluster_tiles), else runs of the context's column order
void make_tiles(Context *ctx, const bsm_pattern_s *PC, int G, int waves, bool cluster, TileSet &ts)
{
    hipStream_t st = ctx->stream;
    const int n = PC->natoms, jt = waves * (64 / PC->b);
    BSM_REQUIRE(G == 2 || G == 4 || G == 8 || G == kMaxRows, BSM_EINVAL, "rows per tile must be 2, 4, 8 or 16");
    BSM_REQUIRE(waves == 1 || (waves == 2 && G <= 8), BSM_EINVAL, "two waves per tile take at most 8 rows");
    const int ng = (n + G - 1) / G;
    ts.G = G;
    ts.waves = waves;
    ts.jt = jt;
    ts.ng = ng;
    ts.groups = DevBuf(ctx, Cut::room(sizeof(int) * ng) + Cut::room(sizeof(int64_t) * (ng + 1)));
    Cut g{ts.groups.as<char>()};
    ts.ntile = g.take<int>(ng);
    ts.toff = g.take<int64_t>(ng + 1);
    k_group_union<<<ng, kPlanThreads, 0, st>>>(n, G, PC->rowptr.as<int>(), PC->cols.as<int>(), jt, ts.ntile);
    int64_t *host = reinterpret_cast<int64_t *>(ctx->host_scalars + kHostCounts);   // counts come back in pinned memory
    k_scan64<<<1, 1024, 0, st>>>(ng, nullptr, ts.toff, host, ts.ntile);
    BSM_HIP_TRY(hipStreamSynchronize(st));
    const int64_t nt = ts.nt = *host;
    BSM_REQUIRE(nt < (int64_t)INT32_MAX, BSM_EINVAL, "too many product tiles");
    ts.hdr = DevBuf(ctx, sizeof(int) * (size_t)std::max<int64_t>(1, nt * (G + G * jt)));
    ts.columns = DevBuf(ctx, Cut::room(sizeof(int) * (size_t)(nt * jt)) + sizeof(int) * (size_t)((5 + G) * nt * jt));
    Cut c{ts.columns.as<char>()};
    ts.tcols = c.take<int>(nt * jt);
    ts.scr = c.take<int>((5 + G) * nt * jt);
    k_group_tiles<<<ng, kPlanThreads, 0, st>>>(n, G, jt, ctx->column_order, PC->rowptr.as<int>(), PC->cols.as<int>(),
                                               ts.toff, nt, ts.hdr.as<int>(), ts.tcols,
                                               ts.scr);
    if (cluster)
        k_cluster_tiles<<<ng, 64, 0, st>>>(n, G, jt, PC->pos.as<double>(), PC->box[0], PC->box[1], PC->box[2],
                                           ts.toff, nt, ts.hdr.as<int>(), ts.tcols,
                                           ts.scr);
    BSM_HIP_TRY(hipGetLastError());
}

// The entry ranges of the plan over `ts`, its flops and its estimated work.
// transposed: plan D = B^T A^T on P_C (C = D^T); the kernel's A operand is B (rows
// over P_B, which is symmetric), its B operand is A.
void count_entries(Context *ctx, const bsm_pattern_s *PA, const bsm_pattern_s *PB, const bsm_pattern_s *PC,
                   const TileSet &ts, int transposed, Plan *plan, EntryCount &ec)
{
    BSM_REQUIRE(!transposed || ts.waves == 1, BSM_EINVAL, "transposed plans use one-wave tiles");
    if (transposed) std::swap(PA, PB);
    hipStream_t st = ctx->stream;
    const int64_t nt = ts.nt;
    plan->G = ts.G;
    plan->waves = ts.waves;
    plan->jt = ts.jt;
    plan->ntiles = nt;
    plan->transposed = transposed;
    plan->ebeg = DevBuf(ctx, sizeof(int64_t) * (size_t)(nt + 1));
    if (nt == 0) BSM_HIP_TRY(hipMemsetAsync(plan->ebeg.ptr, 0, sizeof(int64_t), st));
    if (nt > 0) {
        const size_t places = sizeof(unsigned long long) * kTotalLanes * kTotalStride;
        ec.buf = DevBuf(ctx, places + Cut::room(sizeof(int64_t) * (size_t)nt) + Cut::room(sizeof(int64_t) * (size_t)(nt + 1)));
        Cut c{ec.buf.as<char>()};
        unsigned long long *tri = c.take<unsigned long long>(kTotalLanes * kTotalStride);
        ec.nent = c.take<int64_t>(nt);
        ec.ebeg = c.take<int64_t>(nt + 1);
        BSM_HIP_TRY(hipMemsetAsync(tri, 0, places, st));
        k_tile_entries<0><<<tile_grid(nt), kPlanThreads, 0, st>>>(
            nt, 1, PA->natoms, ts.G, ts.jt, ts.waves, transposed, ts.hdr.as<int>(), ts.tcols,
            PA->rowptr.as<int>(), PA->cols.as<int>(), PA->tmap.as<int>(), PB->rowptr.as<int>(), PB->cols.as<int>(),
            PB->tmap.as<int>(), ec.nent, tri, tri + 1, nullptr, nullptr);
        k_pad_counts<<<(unsigned)((nt + 127) / 128), 128, 0, st>>>(nt, 1, ec.nent);
        int64_t *host = reinterpret_cast<int64_t *>(ctx->host_scalars + kHostCounts);
        k_plan_totals<<<1, kTotalLanes, 0, st>>>(tri, reinterpret_cast<unsigned long long *>(host) + 1);
        k_scan64<<<1, 1024, 0, st>>>(nt, ec.nent, ec.ebeg, host, nullptr);
        k_tile_ebeg<<<(unsigned)((nt + 1 + 127) / 128), 128, 0, st>>>(nt, 1, ec.ebeg,
                                                                      plan->ebeg.as<int64_t>());
        BSM_HIP_TRY(hipStreamSynchronize(st));
        ec.ne = host[0];
        ec.ntri[0] = (unsigned long long)host[1];
        ec.ntri[1] = (unsigned long long)host[2];
    }
    plan->nentries = ec.ne;
    plan->triples = (int64_t)ec.ntri[0];
    plan->rowwork = (int64_t)ec.ntri[1];
    plan->flops = 2.0 * (double)PC->b * PC->b * PC->b * (double)ec.ntri[0];
}

// Write a counted plan's entries; takes the tile headers (and, transposed, moves
// their C slots to (j, i)).
void fill_entries(Context *ctx, const bsm_pattern_s *PA, const bsm_pattern_s *PB, const bsm_pattern_s *PC,
                  TileSet &ts, Plan *plan, const EntryCount &ec)
{
    const int transposed = plan->transposed, es = ts.waves * ts.G + ts.jt;
    if (transposed) std::swap(PA, PB);
    hipStream_t st = ctx->stream;
    const int64_t nt = ts.nt, ne = ec.ne;
    // Groups interleaved by column position share B blocks in L2 while their own A blocks stay
    // there too; four groups of the 16 A class hold 18 MB of A against an XCD's 4 MB, and one group
    // after the other runs better (1000 atoms 20.1 ms against 21.0, 4096 atoms 69.5 against 71.1),
    // while 8 A x 10 A -> 18 A keeps its four (1000 atoms 1.52 ms against 1.54).
    const double group_bytes = (double)ts.G * (double)PA->nnzb / std::max(1, PA->natoms) * PA->b * PA->b * 8.0;
    plan->span = ctx->group_span > 0 ? ctx->group_span : (4.0 * group_bytes > 4.0 * (1 << 20) ? 1 : 4);
    plan->order = DevBuf(ctx, sizeof(int) * (size_t)std::max<int64_t>(1, nt));
    plan->ent = DevBuf(ctx, sizeof(int) * (size_t)((ne + kSpareEntries) * es));
    BSM_HIP_TRY(hipMemsetAsync(plan->ent.as<int>() + ne * es, 0xff, sizeof(int) * kSpareEntries * es, st));
    if (nt > 0) {
        k_tile_order<<<ts.ng, 256, 0, st>>>(ts.ng, plan->span, ts.ntile, ts.toff,
                                            plan->order.as<int>());
        k_tile_entries<1><<<tile_grid(nt), kPlanThreads, 0, st>>>(
            nt, 1, PA->natoms, ts.G, ts.jt, ts.waves, transposed, ts.hdr.as<int>(), ts.tcols,
            PA->rowptr.as<int>(), PA->cols.as<int>(), PA->tmap.as<int>(), PB->rowptr.as<int>(), PB->cols.as<int>(),
            PB->tmap.as<int>(), nullptr, nullptr, nullptr, ec.ebeg, plan->ent.as<int>());
        if (transposed)   // outputs go to the slot of (j, i)
            k_map_cslots<<<(unsigned)((nt + 127) / 128), 128, 0, st>>>(nt, ts.G, ts.jt, PC->tmap.as<int>(),
                                                                       ts.hdr.as<int>());
        BSM_HIP_TRY(hipGetLastError());
    }
    plan->hdr = std::move(ts.hdr);
    BSM_HIP_TRY(hipStreamSynchronize(st));   // before the stages' buffers are freed
}
}  // namespace

void launch_product_f64(Context *ctx, const Plan *plan, double alpha, const bsm_pattern_s *PA,
                        const double *A, const bsm_pattern_s *PB, const double *Bm, double beta,
                        const bsm_pattern_s *PC, double *C)
{
    if (plan->ntiles == 0) return;
    hipStream_t st = ctx->stream;
    Context::ProfRec rec{plan, nullptr, nullptr, BSM_F64};
    if (ctx->profiling) {
        rec.start = ctx->take_event();
        rec.stop = ctx->take_event();
        BSM_HIP_TRY(hipEventRecord(rec.start, st));
    }
    switch (PC->b) {
#define X(b) \
    case b: launch_b<b>(st, plan, A, Bm, C, alpha, beta, ctx->zero_block.as<double>(), 8 * nelems(PA), 8 * nelems(PB)); break;
        BSM_FOR_EACH_B(X)
#undef X
        default: throw Error{BSM_EINVAL, "b must be in 1..16"};
    }
    BSM_HIP_TRY(hipGetLastError());
    if (ctx->profiling) {
        BSM_HIP_TRY(hipEventRecord(rec.stop, st));
        ctx->prof.push_back(rec);
    }
}

// Tiles of 8 rows that P_C takes, counted once per pattern.
static int64_t tiles_of_8(Context *ctx, const bsm_pattern_s *PC)
{
    if (PC->tiles8 >= 0) return PC->tiles8;
    hipStream_t st = ctx->stream;
    const int ng = (PC->natoms + 7) / 8;
    DevBuf buf(ctx, Cut::room(sizeof(int) * ng) + Cut::room(sizeof(int64_t) * (ng + 1)));
    Cut cut{buf.as<char>()};
    int *ntile = cut.take<int>(ng);
    int64_t *toff = cut.take<int64_t>(ng + 1);
    k_group_union<<<ng, kPlanThreads, 0, st>>>(PC->natoms, 8, PC->rowptr.as<int>(), PC->cols.as<int>(), 64 / PC->b,
                                               ntile);
    int64_t *host = reinterpret_cast<int64_t *>(ctx->host_scalars + kHostCounts);
    k_scan64<<<1, 1024, 0, st>>>(ng, nullptr, toff, host, ntile);
    BSM_HIP_TRY(hipStreamSynchronize(st));
    return PC->tiles8 = *host;
}

// Rows per tile of the ring kernels (b = 4 and 9).  8-row tiles copy the fewest blocks per
// triple, but a product of few tiles leaves SIMDs idle behind long serial lists of k, and then
// narrower tiles win: two rows below 1600 tiles of 8 (1.6 per SIMD), four up to about two
// rounds of the resident 8-row waves.  Measured over 75 classes and sizes (64 to 4096 atoms) with
// b = 9 and as many with b = 4, this line is within 2.3% and 0.4% of the best choice in the mean,
// always 8 rows 46% and 51% slower; 64 atoms, b = 9, 8 A: 124 us with 8 rows, 44 with two;
// 512 atoms, 8 A x 6 A -> 14 A: 276 with 8, 232 with four; 1000 atoms, 16 A: 20.2 ms with 8, 22.3 with four.
// Where all three patterns are narrow (mean rows of at most 128 blocks with b = 9, 64 with b = 4: 8 and
// 6 A of silicon) the lists of k are short, a tile's start and end weigh more, and narrower tiles win at
// every count: 1728 atoms, b = 9, 8 A, 706 us with four rows, 617 with two; 4096 atoms, 6 A, 426 with 8,
// 346 with two; 8000 atoms, 8 A, 2979 with 8, 2700 with four; b = 4, 4096 atoms, 6 A, 93 with 8, 75 with
// four.  A wide operand takes that back: 4096 atoms, b = 9, 10 A x 8 A -> 8 A, 1970 with two, 1826 with
// four, 1813 with 8; b = 4, 13824 atoms, 8 A x 6 A -> 8 A, 428 with four, 356 with 8.
static int ring_rows(Context *ctx, const bsm_pattern_s *PA, const bsm_pattern_s *PB, const bsm_pattern_s *PC)
{
    const int64_t nt = tiles_of_8(ctx, PC);
    const int64_t widest = std::max({PA->nnzb, PB->nnzb, PC->nnzb});
    if (nt < 1600) return 2;
    if (widest <= (PC->b == 9 ? 128 : 64) * (int64_t)PC->natoms) return PC->b == 9 && nt < 8000 ? 2 : 4;
    return nt < (PC->b == 9 ? 4000 : 2500) ? 4 : 8;
}

// Rows of a paired launch's plan: its tiles take them twice.
static int pair_rows(Context *ctx, const bsm_pattern_s *PC) { return tiles_of_8(ctx, PC) < 1600 ? 2 : 4; }

static Plan *find_plan(Context *ctx, const bsm_pattern_s *A, const bsm_pattern_s *B, const bsm_pattern_s *C, int variant,
                       int G, int transposed)
{
    auto it = ctx->plans.find(std::make_tuple(A->id, B->id, C->id, variant, G, transposed));
    return it == ctx->plans.end() ? nullptr : it->second.get();
}

// A second plan beside the class's default one: a paired launch's plan, estimated from the class's default plan (about 1.3 times its
// size), fits when free device memory holds twice the estimate and a quarter of the device more.
static bool pair_plan_fits(Context *ctx, const Plan *one)
{
    const double est = 1.3 * (double)(one->ent.bytes + one->hdr.bytes + one->order.bytes + one->ebeg.bytes);
    size_t free_b = 0, total_b = 0;
    BSM_HIP_TRY(hipMemGetInfo(&free_b, &total_b));
    return (double)free_b >= 2.0 * est + std::max(8.0 * (1u << 30), 0.25 * (double)total_b);
}

Plan *get_pair_plan(Context *ctx, const bsm_pattern_s *PA, const bsm_pattern_s *PB, const bsm_pattern_s *PC)
{
    const int b = PC->b;
    if (b != 4 && b != 9) return nullptr;
    if (ctx->product_variant >= 0 && ctx->product_variant != 4) return nullptr;
    // direct ring plan of half the paired tile's rows
    const int G = pair_rows(ctx, PC);
    if (Plan *p = find_plan(ctx, PA, PB, PC, 4, G, 0)) return p;
    // The 4-row plan is a second plan beside the default one (about 1.3 times its size, 4.9 GB
    // for the 16 A class at 4096 atoms, eight times that at 32768): built only while free
    // device memory holds twice that and a quarter of the device besides (room for what the
    // caller allocates next), else the pair runs as two launches (same results either way)
    if (!pair_plan_fits(ctx, get_plan(ctx, PA, PB, PC))) return nullptr;
    return get_plan_kind(ctx, PA, PB, PC, 4, G);
}

namespace {
template <int B, int G, int TR>
void launch_pair_g(hipStream_t st, const Plan *plan, const double *A, const double *A2, const double *Bm, double *C,
                 double *C2, double alpha, double beta, const double *zblk, int64_t a_bytes, int64_t b_bytes)
{
    const int64_t nwg_padded = ((plan->ntiles + kXcd - 1) / kXcd) * kXcd;
    const bool buf = a_bytes <= (int64_t)kBufMaxBytes && b_bytes <= (int64_t)kBufMaxBytes;
    auto go = [&](auto kern, bool rs) {
        kern<<<(unsigned)nwg_padded, 64, 0, st>>>(
            plan->ntiles, nwg_padded, plan->order.as<int>(), plan->hdr.as<int>(), plan->ebeg.as<int64_t>(),
            plan->ent.as<int>(), A, A2, Bm, zblk, C, C2, alpha, beta, rs ? (unsigned)a_bytes : 0u,
            rs ? (unsigned)a_bytes : 0u, rs ? (unsigned)b_bytes : 0u);
    };
    if constexpr (B == 4) {
        if (can_pack(A, A2, Bm)) {
            if (buf) go(k_product_ring_pair<B, G, kPackedPairDepth, kPackedBuffers, TR>, true);
            else go(k_product_ring_pair<B, G, kPackedPairDepth, kPackedCopies, TR>, false);
            return;
        }
    }
    if (buf) go(k_product_ring_pair<B, G, 2, kBufferCopies, TR>, true);
    else go(k_product_ring_pair<B, G, 2, kPointerCopies, TR>, false);
}
template <int B, int TR>
void launch_pair(hipStream_t st, const Plan *plan, const double *A, const double *A2, const double *Bm, double *C,
                 double *C2, double alpha, double beta, const double *zblk, int64_t a_bytes, int64_t b_bytes)
{
    if (plan->G == 2) launch_pair_g<B, 4, TR>(st, plan, A, A2, Bm, C, C2, alpha, beta, zblk, a_bytes, b_bytes);
    else launch_pair_g<B, 8, TR>(st, plan, A, A2, Bm, C, C2, alpha, beta, zblk, a_bytes, b_bytes);
}
}  // namespace

void launch_product_pair_f64(Context *ctx, const Plan *plan, double alpha, const bsm_pattern_s *PA,
                             const double *A, const double *A2, const bsm_pattern_s *PB, const double *Bm,
                             double beta, const bsm_pattern_s *PC, double *C, double *C2)
{
    BSM_REQUIRE(plan->variant == 4 && (plan->G == 2 || plan->G == 4) && !plan->transposed && (PC->b == 4 || PC->b == 9),
                BSM_EINVAL, "a paired launch takes a direct 2- or 4-row ring plan, b = 4 or 9");
    if (plan->ntiles == 0) return;
    hipStream_t st = ctx->stream;
    Context::ProfRec rec{plan, nullptr, nullptr, BSM_F64, 2};
    if (ctx->profiling) {
        rec.start = ctx->take_event();
        rec.stop = ctx->take_event();
        BSM_HIP_TRY(hipEventRecord(rec.start, st));
    }
    const int64_t ab = 8 * nelems(PA), bb = 8 * nelems(PB);
    if (PC->b == 9)
        launch_pair<9, 0>(st, plan, A, A2, Bm, C, C2, alpha, beta, ctx->zero_block.as<double>(), ab, bb);
    else
        launch_pair<4, 0>(st, plan, A, A2, Bm, C, C2, alpha, beta, ctx->zero_block.as<double>(), ab, bb);
    BSM_HIP_TRY(hipGetLastError());
    if (ctx->profiling) {
        BSM_HIP_TRY(hipEventRecord(rec.stop, st));
        ctx->prof.push_back(rec);
    }
}

Plan *get_pair_plan_a(Context *ctx, const bsm_pattern_s *PA, const bsm_pattern_s *PB, const bsm_pattern_s *PC)
{
    const int b = PC->b;
    if (b != 4 && b != 9) return nullptr;
    if (ctx->product_variant >= 0 && ctx->product_variant != 4) return nullptr;
    // transposed ring plan: the tiles' rows walk B and B2, the shared A is the copied operand
    const int G = pair_rows(ctx, PC);
    if (Plan *p = find_plan(ctx, PA, PB, PC, 4, G, 2)) return p;
    if (!pair_plan_fits(ctx, get_plan(ctx, PA, PB, PC))) return nullptr;
    return get_transposed_plan(ctx, PA, PB, PC, G);
}

void launch_product_pair_a_f64(Context *ctx, const Plan *plan, double alpha, const bsm_pattern_s *PA,
                               const double *A, const bsm_pattern_s *PB, const double *Bm, const double *B2,
                               double beta, const bsm_pattern_s *PC, double *C, double *C2)
{
    BSM_REQUIRE(plan->variant == 4 && (plan->G == 2 || plan->G == 4) && plan->transposed && (PC->b == 4 || PC->b == 9),
                BSM_EINVAL, "a paired launch sharing A takes a transposed 2- or 4-row ring plan, b = 4 or 9");
    if (plan->ntiles == 0) return;
    hipStream_t st = ctx->stream;
    Context::ProfRec rec{plan, nullptr, nullptr, BSM_F64, 2};
    if (ctx->profiling) {
        rec.start = ctx->take_event();
        rec.stop = ctx->take_event();
        BSM_HIP_TRY(hipEventRecord(rec.start, st));
    }
    // the kernel's row operand is B (and B2), its column operand the shared A
    const int64_t ab = 8 * nelems(PB), bb = 8 * nelems(PA);
    if (PC->b == 9)
        launch_pair<9, 1>(st, plan, Bm, B2, A, C, C2, alpha, beta, ctx->zero_block.as<double>(), ab, bb);
    else
        launch_pair<4, 1>(st, plan, Bm, B2, A, C, C2, alpha, beta, ctx->zero_block.as<double>(), ab, bb);
    BSM_HIP_TRY(hipGetLastError());
    if (ctx->profiling) {
        BSM_HIP_TRY(hipEventRecord(rec.stop, st));
        ctx->prof.push_back(rec);
    }
}

void launch_product_mixed(Context *ctx, const Plan *plan, int prec, double alpha, const bsm_pattern_s *PA,
                          const double *A, const bsm_pattern_s *PB, const double *Bm, double beta,
                          const bsm_pattern_s *PC, double *C)
{
    if (prec == BSM_F64) {
        launch_product_f64(ctx, plan, alpha, PA, A, PB, Bm, beta, PC, C);
        return;
    }
    BSM_REQUIRE(prec == BSM_F32 || prec == BSM_BF16, BSM_EINVAL, "precision must be F64, F32 or BF16");
    if (plan->G > 8) plan = get_plan_kind(ctx, PA, PB, PC, 0, default_rows_per_wave(PC->b));   // wave tiles
    if (plan->variant == 6) plan = get_plan_kind(ctx, PA, PB, PC, 4, plan->G);   // reduced precision: the ring
    // BF16 on the matrix cores for products of two matrices on one pattern (the wide 16 A class,
    // where the dense MFMA tiles pay); the narrower classes run faster on the FP32 VALU ring with
    // BF16-rounded operands, on their own (possibly transposed) plans
    const bool mfma = prec == BSM_BF16 && PC->b == 9 && PA == PB;
    if (mfma && (plan->variant == 5 || plan->transposed))
        plan = get_plan_kind(ctx, PA, PB, PC, 4, plan->G);   // the matrix cores take direct one-wave tiles
    if (plan->ntiles == 0) return;
    hipStream_t st = ctx->stream;
    if (mfma && (plan->G == 4 || plan->G == 8) && (plan->variant == 3 || plan->variant == 4)) {
        // matrix cores: operands packed to BF16 (B transposed), FP32 accumulation
        unsigned short *pa = reinterpret_cast<unsigned short *>(ctx->scratch_f32(0, PA->nnzb * (kPackedBlock / 2)));
        unsigned short *pb = reinterpret_cast<unsigned short *>(ctx->scratch_f32(1, PB->nnzb * (kPackedBlock / 2)));
        k_pack_bf16_blocks<<<dim3((unsigned)((PA->nnzb + kPackBlocks - 1) / kPackBlocks), 2), kPackThreads, 0, st>>>(
            PA->nnzb, A, Bm, pa, pb);   // one pattern
        Context::ProfRec rec{plan, nullptr, nullptr, prec};
        if (ctx->profiling) {
            rec.start = ctx->take_event();
            rec.stop = ctx->take_event();
            BSM_HIP_TRY(hipEventRecord(rec.start, st));
        }
        const int64_t nwg_padded = ((plan->ntiles + kXcd - 1) / kXcd) * kXcd;
        // variant 4: buffer copies while the packed operands fit a buffer resource
        const int64_t ab = PA->nnzb * (int64_t)kPackedBytes, bb = PB->nnzb * (int64_t)kPackedBytes;
        const bool buf = plan->variant == 4 && ab <= (int64_t)kBufMaxBytes && bb <= (int64_t)kBufMaxBytes;
        auto go = [&](auto kern) {
            kern<<<(unsigned)nwg_padded, 64, 0, st>>>(plan->ntiles, nwg_padded, plan->order.as<int>(),
                                                      plan->hdr.as<int>(), plan->ebeg.as<int64_t>(),
                                                      plan->ent.as<int>(), pa, pb,
                                                      ctx->zero_block.as<unsigned short>(), C, alpha, beta,
                                                      buf ? (unsigned)ab : 0u, buf ? (unsigned)bb : 0u);
        };
        if (plan->G == 8)
            buf ? go(k_product_mfma_bf16<8, true>) : go(k_product_mfma_bf16<8, false>);
        else
            buf ? go(k_product_mfma_bf16<4, true>) : go(k_product_mfma_bf16<4, false>);
        BSM_HIP_TRY(hipGetLastError());
        if (ctx->profiling) {
            BSM_HIP_TRY(hipEventRecord(rec.stop, st));
            ctx->prof.push_back(rec);
        }
        return;
    }
    const int64_t na = nelems(PA), nb = nelems(PB);
    float *a32 = ctx->scratch_f32(0, na), *b32 = ctx->scratch_f32(1, nb);
    const int bf = prec == BSM_BF16 ? 1 : 0;
    k_round_copy<<<(unsigned)((na + 255) / 256), 256, 0, st>>>(na, A, a32, bf);
    k_round_copy<<<(unsigned)((nb + 255) / 256), 256, 0, st>>>(nb, Bm, b32, bf);
    Context::ProfRec rec{plan, nullptr, nullptr, prec};
    if (ctx->profiling) {
        rec.start = ctx->take_event();
        rec.stop = ctx->take_event();
        BSM_HIP_TRY(hipEventRecord(rec.start, st));
    }
    switch (PC->b) {
#define X(b) \
    case b: launch_b32<b>(st, plan, a32, b32, C, alpha, beta, ctx->zero_block.as<float>(), 4 * na, 4 * nb); break;
        BSM_FOR_EACH_B(X)
#undef X
        default: throw Error{BSM_EINVAL, "b must be in 1..16"};
    }
    BSM_HIP_TRY(hipGetLastError());
    if (ctx->profiling) {
        BSM_HIP_TRY(hipEventRecord(rec.stop, st));
        ctx->prof.push_back(rec);
    }
}

// Estimated cost of a plan for the ring kernels: rows multiplied plus the
// fixed work of an entry (copies, waits, B reads), worth some 4.5 rows as measured
// on b = 9 entries of 8 rows.  It picks well for the others too: over 136 classes
// of 216 to 1000 atoms, b = 4, 5, 9 and 13, the plan it takes is 0.1% slower than
// the better of direct and transposed in the mean, and by more than 1% in two
// (512 atoms, b = 13, 10 A x 8 A -> 16 A 2.76 ms, 2.54 transposed).
static double plan_cost(const Plan *p) { return (double)p->rowwork + 4.5 * (double)p->nentries; }

static std::unique_ptr<Plan> named_plan(const bsm_pattern_s *A, const bsm_pattern_s *B, const bsm_pattern_s *C,
                                        int variant)
{
    std::unique_ptr<Plan> plan(new Plan());
    plan->ids[0] = A->id;
    plan->ids[1] = B->id;
    plan->ids[2] = C->id;
    plan->cutoffs[0] = A->cutoff;
    plan->cutoffs[1] = B->cutoff;
    plan->cutoffs[2] = C->cutoff;
    plan->natoms = C->natoms;
    plan->b = C->b;
    plan->variant = variant;
    return plan;
}

// Whether tiles of near columns serve a plan whose kernel walks rows of PA and reads
// columns of PB: where the columns' own range cuts many k (its radius well below those of
// the rows and outputs together).  Where it cuts few or none (a narrow matrix times a wide
// one, 6 A x 16 A -> 10 A), a tile's k are its rows' k and the row-set order idles fewer
// lanes: there counted cost 0.478 against 0.509 of the clustered tiles, against 0.426 and
// 0.384 for 16 A x 16 A -> 16 A.  Nor does any k fall to the columns of a fuller PB, sooner so with
// few rows to a tile.  b = 9, row sets and near columns: 4 rows, 0.38 full, 717 and 773 us (512
// atoms, 10 A); paired, 0.59 full, 21.4 and 21.9 ms, 0.77 full, 37.7 and 38.9 (1000 atoms, 14 and
// 16 A), 0.21 full, 134.3 and 130.3 (4096 atoms, 16 A); 2 rows, 0.50 full, 135.5 and 140.0 us, 0.21
// full, 37.4 and 35.5 (216 atoms, 8 and 6 A); 8 rows, 0.59 full, 12.42 and 12.00 ms, 0.77 full,
// 20.4 and 20.7.  b = 4 draws the second line at any rows (4 rows, 0.38 full, 142 and 133 us: 512
// atoms, 12 A x 10 A -> 10 A; 8 rows, 0.77 full, 2.19 and 2.25 ms: 1000 atoms, 16 A), and the other
// b's fewer columns a later one (480 atoms, b = 13, 10 A x 6 A -> 16 A, 0.40 full, 957 and 928 us).
static bool cluster_pays(const bsm_pattern_s *PA, const bsm_pattern_s *PB, const bsm_pattern_s *PC, int G)
{
    const double n = (double)PB->natoms;
    const double full = PC->b != 4 && PC->b != 9 ? 0.8 : PC->b == 9 && G <= 4 ? 0.35 : 0.7;
    return PA->cutoff + PC->cutoff - PB->cutoff >= 0.3 * PC->cutoff && (double)PB->nnzb < full * n * n;
}

// direct, transposed, or (both) the one with the smaller estimated cost: both are
// counted, one is written.
static std::unique_ptr<Plan> new_plan(Context *ctx, const bsm_pattern_s *A, const bsm_pattern_s *B,
                                      const bsm_pattern_s *C, int variant, int G, bool direct, bool transposed)
{
    TileSet tiles[2];   // plain, clustered
    std::unique_ptr<Plan> plan;
    EntryCount ec;
    TileSet *used = nullptr;
    for (int tr = direct ? 0 : 1; tr <= (transposed ? 1 : 0); ++tr) {
        const bool near = variant == 4 && ctx->column_order == 1 && (tr ? cluster_pays(B, A, C, G) : cluster_pays(A, B, C, G));
        TileSet &ts = tiles[near ? 1 : 0];
        if (ts.G == 0) make_tiles(ctx, C, G, variant == 5 ? 2 : 1, near, ts);
        std::unique_ptr<Plan> p = named_plan(A, B, C, variant);
        EntryCount e;
        count_entries(ctx, A, B, C, ts, tr, p.get(), e);
        if (plan && !(plan_cost(p.get()) < plan_cost(plan.get()))) continue;
        plan = std::move(p);
        ec = std::move(e);
        used = &ts;
    }
    fill_entries(ctx, A, B, C, *used, plan.get(), ec);
    return plan;
}

Plan *get_transposed_plan(Context *ctx, const bsm_pattern_s *A, const bsm_pattern_s *B, const bsm_pattern_s *C, int G)
{
    auto key = std::make_tuple(A->id, B->id, C->id, 4, G, 2);
    auto it = ctx->plans.find(key);
    if (it != ctx->plans.end()) return it->second.get();
    std::unique_ptr<Plan> plan = new_plan(ctx, A, B, C, 4, G, false, true);
    Plan *raw = plan.get();
    ctx->plans[key] = std::move(plan);
    return raw;
}

Plan *get_plan_kind(Context *ctx, const bsm_pattern_s *A, const bsm_pattern_s *B, const bsm_pattern_s *C,
                    int variant, int G, bool allow_transposed)
{
    // C = (B^T A^T)^T is an option for the default ring kernel when A and B lie on
    // different patterns (all patterns are symmetric): a wide A times a narrow B
    // then walks the narrow pattern, with far fewer idle lanes
    const bool try_t = allow_transposed && ctx->transposed_plans > 0 && variant == 4 && G <= 8 &&
                       (C->b == 4 || C->b == 9 || any_b_ring(C->b)) && A->id != B->id;
    auto key = std::make_tuple(A->id, B->id, C->id, variant, G, try_t ? 1 : 0);
    auto it = ctx->plans.find(key);
    if (it != ctx->plans.end()) return it->second.get();
    std::unique_ptr<Plan> plan = new_plan(ctx, A, B, C, variant, G, !(try_t && ctx->transposed_plans == 2), try_t);
    Plan *raw = plan.get();
    ctx->plans[key] = std::move(plan);
    return raw;
}

Plan *get_plan(Context *ctx, const bsm_pattern_s *A, const bsm_pattern_s *B, const bsm_pattern_s *C, int prec)
{
    int variant = ctx->product_variant >= 0 ? ctx->product_variant : default_variant(C->b);
    if (variant == 6 && C->b != 9) variant = 4;   // the FP64 matrix-core tiles are for b = 9
    // other b: the ring kernels of product_any_b.h by default, their row count and operands they
    // can address; else the scalar-operand kernel (which any explicit variant from 2 on means too)
    if (C->b != 9 && C->b != 4) {
        if (ctx->product_variant < 0 && ctx->rows_per_wave == 0 && any_b_ring(C->b) && fits_buffers(A, B))
            return get_plan_kind(ctx, A, B, C, 4, any_b_rows(C->b, tiles_of_8(ctx, C) < 1600), true);
        if (variant >= 2) variant = 0;
    }
    int G = variant == 2 ? kMaxRows : (ctx->rows_per_wave > 0 ? ctx->rows_per_wave : default_rows_per_wave(C->b));
    if ((variant == 4 || variant == 5 || variant == 6) && (C->b == 4 || C->b == 9) && ctx->rows_per_wave == 0)
        G = variant == 4 && !(prec == BSM_BF16 && C->b == 9 && A == B) ? ring_rows(ctx, A, B, C) : 8;
    if ((variant == 5 || variant == 6) && G < 4) G = 4;   // two-wave and matrix-core tiles take 4 or 8 rows
    return get_plan_kind(ctx, A, B, C, variant, G, true);
}

}  // namespace bsm
