// Learned initial guess: pair descriptors, a three-layer perceptron with FP32
// training kernels and BF16 matrix-core inference, Adam, and block predictions.
//
// The network maps the 32-value descriptor of an atom pair to a b x b block
// correction of the Hotelling or LNV start (include/bsm_guess.h).  Its
// workload is small next to the block products (about 58 kFLOP per pair per
// forward pass), so the kernels aim at plain, deterministic data flow:
//   - training: tiles of 16 samples run forward and backward on the FP32 matrix
//     cores, weight gradients are contractions over ranges of samples, and a
//     fixed-order reduction adds the ranges (no atomics);
//   - inference (BF16): each wavefront pushes 16 samples through the three
//     layers with 16x16x16 BF16 MFMAs (FP32 accumulation), weights pre-packed
//     into the per-lane operand layout and kept in LDS, activations in registers.
#include "bsm_internal.h"
#include "bsm_guess.h"

#include <cmath>
#include <vector>

namespace bsm {
namespace {

constexpr int kD = BSM_DESC_DIM;    // descriptor length
constexpr int kH = BSM_MLP_WIDTH;   // hidden width
constexpr int kTS = 32;             // samples per training tile
constexpr int kNT = 256;            // threads per workgroup

struct Offs {
    int64_t w1, b1, w2, b2, w3, b3, total;
};

__host__ __device__ inline Offs offsets(int M)
{
    Offs o;
    o.w1 = 0;
    o.b1 = (int64_t)kD * kH;
    o.w2 = o.b1 + kH;
    o.b2 = o.w2 + (int64_t)kH * kH;
    o.w3 = o.b2 + kH;
    o.b3 = o.w3 + (int64_t)kH * M;
    o.total = o.b3 + M;
    return o;
}

// Where a forward pass puts its outputs: Y[s][o], or FP64 blocks
// blocks[s][o] <- beta blocks[s][o] + scale y (beta == 0 overwrites).
struct Out {
    float *Y;
    double *blocks;
    double scale, beta;
};

__device__ inline void put(const Out &out, int64_t at, float y)
{
    if (out.Y) {
        out.Y[at] = y;
    } else {
        const double v = out.scale * (double)y;
        out.blocks[at] = out.beta == 0.0 ? v : out.beta * out.blocks[at] + v;
    }
}

// ------------------------------------------------------------------ descriptors

// orders a wavefront's own shared-memory accesses across its lanes
__device__ inline void wave_sync()
{
    __builtin_amdgcn_fence(__ATOMIC_ACQ_REL, "wavefront");
    __builtin_amdgcn_wave_barrier();
}

__device__ inline double dmul(double a, double b) { return __dmul_rn(a, b); }
__device__ inline double dadd(double a, double b) { return __dadd_rn(a, b); }

__device__ inline void min_image(const double *__restrict__ pos, double3 box, int i, int j, double r[3])
{
    const double bx[3] = {box.x, box.y, box.z};
#pragma unroll
    for (int c = 0; c < 3; ++c) {
        const double d = pos[3 * j + c] - pos[3 * i + c];
        r[c] = d - dmul(bx[c], rint(d / bx[c]));
    }
}

__device__ inline double norm2(const double r[3]) { return dadd(dadd(dmul(r[0], r[0]), dmul(r[1], r[1])), dmul(r[2], r[2])); }

// tetrahedral directions of the first diamond sublattice, before the 1 / sqrt 3
__constant__ double kTetra[4][3] = {{1, 1, 1}, {1, -1, -1}, {-1, 1, -1}, {-1, -1, 1}};

constexpr int kFrame = 24;   // doubles per atom frame
constexpr double kBond0 = 2.3512589712747505;   // 5.43 sqrt(3) / 4 rounded to FP64: the ideal Si-Si bond, Angstrom
// environment density of an ideal-lattice atom over a 6 A neighbour pattern: the five
// diamond shells inside 6 A (4, 12, 12, 6, 12 atoms at 5.43 sqrt(q) / 4 A, q = 3, 8, 11,
// 16, 19) weighted by exp(-d / 1.5 A)
constexpr double kRho0 = 2.751647885181917;

constexpr int kFrameAtoms = 16;   // atoms of a workgroup
constexpr int kFrameLanes = 16;   // lanes of an atom

// Per atom (see the header): fr[24 i] = s, fr[24 i + 1 + 3 a + c] = e[a][c],
// fr[24 i + 13 + a] = l[a], fr[24 i + 17 + c] = c_i[c], fr[24 i + 20] = rho_i (the
// sum over the row's other atoms of exp(-d / 1.5 A), in column order).
// Sixteen lanes per atom, a neighbour each at a time: distances and exponentials side by side, the sum in column
// order from LDS, and the nearest four by the rank of every neighbour among the sixteen and the four kept so far
// (by distance, then index; empty places are (infinity, INT_MAX)).  4096 atoms, 6 A rows: 18 us, against
// 107 with a thread for all of an atom's neighbours and 40 with one lane of an atom walking the list.
__global__ __launch_bounds__(kFrameAtoms * kFrameLanes) void k_atom_frames(int n, const double *__restrict__ pos,
                                                                           double3 box, const int *__restrict__ rowptr,
                                                                           const int *__restrict__ cols,
                                                                           double *__restrict__ fr,
                                                                           int *__restrict__ bad)
{
    constexpr int L = kFrameLanes;
    __shared__ double sd[kFrameAtoms][L + 4], sx[kFrameAtoms][L], sr[kFrameAtoms][4][3];   // the kept ones last
    __shared__ int sj[kFrameAtoms][L + 4];
    const int w = threadIdx.x / L, l = threadIdx.x % L;
    const int i = blockIdx.x * kFrameAtoms + w;
    if (i >= n) return;   // no workgroup barriers below
    if (l < 4) {
        sd[w][L + l] = INFINITY;
        sj[w][L + l] = INT_MAX;
        for (int c = 0; c < 3; ++c) sr[w][l][c] = 0.0;
    }
    int found = 0;
    double rho = 0.0;
    const int end = rowptr[i + 1];
    for (int s0 = rowptr[i]; s0 < end; s0 += L) {
        double r[3] = {0.0, 0.0, 0.0}, d2 = INFINITY, x = 0.0;
        int j = s0 + l < end ? cols[s0 + l] : i;
        if (j != i) {
            ++found;
            min_image(pos, box, i, j, r);
            d2 = norm2(r);
            x = exp(-sqrt(d2) / 1.5);
        }
        if (j == i || !(d2 == d2)) {   // not a neighbour to choose
            d2 = INFINITY;
            j = INT_MAX;
        }
        wave_sync();   // the neighbours before have been read, the kept ones written
        sd[w][l] = d2;
        sj[w][l] = j;
        sx[w][l] = x;
        wave_sync();
        // rank of this lane's neighbour, and in the first four lanes of a kept one
        const double k2 = sd[w][L + (l & 3)];
        const int kj = sj[w][L + (l & 3)];
        double kr[3];
        for (int c = 0; c < 3; ++c) kr[c] = sr[w][l & 3][c];
        int rank = 0, krank = 0;
#pragma unroll
        for (int q = 0; q < L + 4; ++q) {
            const double e2 = sd[w][q];
            const int ej = sj[w][q];
            rank += e2 < d2 || (e2 == d2 && ej < j);
            krank += e2 < k2 || (e2 == k2 && ej < kj);
            if (q < L) rho = dadd(rho, sx[w][q]);
        }
        wave_sync();   // all ranks known: the first four become the kept ones
        if (j != INT_MAX && rank < 4) {
            sd[w][L + rank] = d2;
            sj[w][L + rank] = j;
            for (int c = 0; c < 3; ++c) sr[w][rank][c] = r[c];
        }
        if (l < 4 && kj != INT_MAX && krank < 4) {
            sd[w][L + krank] = k2;
            sj[w][L + krank] = kj;
            for (int c = 0; c < 3; ++c) sr[w][krank][c] = kr[c];
        }
    }
    for (int off = L / 2; off > 0; off >>= 1) found += __shfl_xor(found, off, 64);
    wave_sync();
    if (l != 0) return;
    double bd[4], bv[4][3];
#pragma unroll
    for (int q = 0; q < 4; ++q) {
        bd[q] = sd[w][L + q];
        for (int c = 0; c < 3; ++c) bv[q][c] = sr[w][q][c];
    }
    if (found < 4) {
        *bad = 1;
        return;
    }
    const double inv3 = 1.0 / sqrt(3.0);
    double u[4][3], dots[4][4];
    for (int q = 0; q < 4; ++q) {
        const double d = sqrt(bd[q]);
        for (int c = 0; c < 3; ++c) u[q][c] = bv[q][c] / d;
        for (int a = 0; a < 4; ++a)
            dots[q][a] = dadd(dadd(dmul(u[q][0], kTetra[a][0] * inv3), dmul(u[q][1], kTetra[a][1] * inv3)),
                              dmul(u[q][2], kTetra[a][2] * inv3));
    }
    double sA = 0.0, sB = 0.0;
    for (int q = 0; q < 4; ++q) {
        double mA = -INFINITY, mB = -INFINITY;
        for (int a = 0; a < 4; ++a) {
            mA = fmax(mA, dots[q][a]);
            mB = fmax(mB, -dots[q][a]);
        }
        sA = dadd(sA, mA);
        sB = dadd(sB, mB);
    }
    const double sg = sA >= sB ? 1.0 : -1.0;
    double *f = fr + kFrame * (int64_t)i;
    f[0] = sg;
    for (int a = 0; a < 4; ++a) {
        int best = 0;
        for (int q = 1; q < 4; ++q)
            if (sg * dots[q][a] > sg * dots[best][a]) best = q;
        for (int c = 0; c < 3; ++c) f[1 + 3 * a + c] = u[best][c];
        f[13 + a] = sqrt(bd[best]);
    }
    for (int c = 0; c < 3; ++c) f[17 + c] = dadd(dadd(dadd(bv[0][c], bv[1][c]), bv[2][c]), bv[3][c]) / 4.0;
    f[20] = rho;
}

constexpr int kDescSlots = 128;   // threads of k_pair_desc

// A thread per slot; a workgroup's descriptors, contiguous in memory, go through LDS into whole lines (43 us
// for 856 thousand slots, 110 MB written, against 54 with each thread storing its own 128 bytes).
__global__ __launch_bounds__(kDescSlots) void k_pair_desc(int64_t nnz, const int *__restrict__ rowidx, const int *__restrict__ cols,
                            const double *__restrict__ pos, double3 box, double rc, const double *__restrict__ fr,
                            float *__restrict__ X)
{
    __shared__ float sv[kDescSlots][kD + 1];
    const int64_t s0 = (int64_t)blockIdx.x * kDescSlots;
    const int64_t s = min(s0 + threadIdx.x, nnz - 1);   // threads past the end repeat the last slot
    const int i = rowidx[s], j = cols[s];
    double r[3];
    min_image(pos, box, i, j, r);
    const double d = sqrt(norm2(r));
    double rh[3];
    for (int c = 0; c < 3; ++c) rh[c] = d > 0.0 ? r[c] / d : 0.0;
    const double *fi = fr + kFrame * (int64_t)i, *fj = fr + kFrame * (int64_t)j;
    float v[kD];
    for (int c = 0; c < 3; ++c) v[c] = (float)(r[c] / rc);
    v[3] = (float)(d / rc);
    v[4] = (float)(dmul(d / rc, d / rc));
    v[5] = (float)exp(-d / 1.5);
    v[6] = (float)fi[0];
    v[7] = (float)fj[0];
    for (int a = 0; a < 4; ++a) {
        v[8 + a] = (float)dadd(dadd(dmul(rh[0], fi[1 + 3 * a]), dmul(rh[1], fi[2 + 3 * a])), dmul(rh[2], fi[3 + 3 * a]));
        v[12 + a] = (float)dadd(dadd(dmul(rh[0], fj[1 + 3 * a]), dmul(rh[1], fj[2 + 3 * a])), dmul(rh[2], fj[3 + 3 * a]));
        v[16 + a] = (float)(10.0 * (fi[13 + a] - kBond0));
        v[20 + a] = (float)(10.0 * (fj[13 + a] - kBond0));
    }
    for (int c = 0; c < 3; ++c) {
        v[24 + c] = (float)(10.0 * fi[17 + c]);
        v[27 + c] = (float)(10.0 * fj[17 + c]);
    }
    v[30] = (float)(10.0 * (fi[20] - kRho0));
    v[31] = (float)(10.0 * (fj[20] - kRho0));
    for (int q = 0; q < kD; ++q) sv[threadIdx.x][q] = v[q];
    __syncthreads();
    float4 *o = reinterpret_cast<float4 *>(X + (int64_t)kD * s0);
    const int cnt = (int)min((int64_t)kDescSlots, nnz - s0) * (kD / 4);
    for (int e = threadIdx.x; e < cnt; e += kDescSlots) {
        const float *q = &sv[e / (kD / 4)][e % (kD / 4) * 4];
        o[e] = make_float4(q[0], q[1], q[2], q[3]);
    }
}

// ------------------------------------------------------------------ FP32 network

__device__ inline double wave_sum(double x)
{
    for (int off = 32; off > 0; off >>= 1) x += __shfl_xor(x, off, 64);
    return x;
}

// Forward pass over samples 0..n-1: thread t serves hidden / output unit o = t % 128 for
// samples of its half (t / 128) of a 32-sample tile.
__global__ __launch_bounds__(kNT) void k_mlp_f32(const float *__restrict__ prm, int M, int64_t n,
                                                 const float *__restrict__ X, Out out)
{
    __shared__ float xs[kTS][kD];
    __shared__ float a1[kTS][kH];
    __shared__ float a2[kTS][kH];
    const Offs of = offsets(M);
    const float *W1 = prm + of.w1, *B1 = prm + of.b1, *W2 = prm + of.w2, *B2 = prm + of.b2, *W3 = prm + of.w3,
                *B3 = prm + of.b3;
    const int t = threadIdx.x, o = t & (kH - 1), half = t >> 7, sb = half * (kTS / 2);
    const int64_t ntiles = (n + kTS - 1) / kTS;
    for (int64_t tile = blockIdx.x; tile < ntiles; tile += gridDim.x) {
        const int64_t s0 = tile * kTS;
        const int cnt = (int)min((int64_t)kTS, n - s0);
        for (int e = t; e < kTS * kD; e += kNT) {
            const int s = e / kD, k = e % kD;
            float v = 0.f;
            if (s < cnt) {
                v = X[(s0 + s) * kD + k];
            }
            xs[s][k] = v;
        }
        __syncthreads();
        float acc[16];
        {
            const float bb = B1[o];
#pragma unroll
            for (int s = 0; s < 16; ++s) acc[s] = bb;
#pragma unroll 4
            for (int k = 0; k < kD; ++k) {
                const float w = W1[k * kH + o];
#pragma unroll
                for (int s = 0; s < 16; ++s) acc[s] = fmaf(xs[sb + s][k], w, acc[s]);
            }
#pragma unroll
            for (int s = 0; s < 16; ++s) a1[sb + s][o] = tanhf(acc[s]);
        }
        __syncthreads();
        {
            const float bb = B2[o];
#pragma unroll
            for (int s = 0; s < 16; ++s) acc[s] = bb;
#pragma unroll 4
            for (int k = 0; k < kH; ++k) {
                const float w = W2[k * kH + o];
#pragma unroll
                for (int s = 0; s < 16; ++s) acc[s] = fmaf(a1[sb + s][k], w, acc[s]);
            }
#pragma unroll
            for (int s = 0; s < 16; ++s) a2[sb + s][o] = tanhf(acc[s]);
        }
        __syncthreads();
        if (o < M) {
            const float bb = B3[o];
#pragma unroll
            for (int s = 0; s < 16; ++s) acc[s] = bb;
#pragma unroll 4
            for (int k = 0; k < kH; ++k) {
                const float w = W3[k * M + o];
#pragma unroll
                for (int s = 0; s < 16; ++s) acc[s] = fmaf(a2[sb + s][k], w, acc[s]);
            }
        }
        if (o < M)
            for (int s = 0; s < 16; ++s)
                if (sb + s < cnt) put(out, (s0 + sb + s) * M + o, acc[s]);
        // the next tile's first barrier orders the LDS reuse
    }
}

// ------------------------------------------------------------------ FP32 gradients
// A minibatch's gradient in three launches over FP32 matrix cores: k_mlp_backprop runs
// tiles of 16 samples forward and backward and keeps every layer's activations and
// errors (n x 600 floats, resident in L2), k_mlp_wgrad contracts them over the samples
// into partial gradients of kSplits sample ranges, k_sum_gradient adds the partials in
// order.  The former kernel did all of it in one pass of 32-sample tiles on the vector
// units, with a shared-memory read per fused multiply-add and a gradient row of 31
// thousand floats per workgroup to write and add up: 85 + 31 + 8 us (forward and backward,
// sum of the rows, loss by one thread) for 4096 samples and 81 outputs, on 128 of the 256
// CUs, and 152 us a call; these take 20 + 12 + 4, and the call 43.  The products need 5 us
// at the FP32 matrix rate: what is left is five layers' latency, each a row of loads,
// products, a tanh and a barrier, with one workgroup per CU, and the way of the
// activations through memory to the second launch.
constexpr int kGS = 16;            // samples of a tile
constexpr int kGradChunk = 8192;   // samples whose activations are held at once
constexpr int kSplits = 32;        // sample ranges of the weight gradients, at most
constexpr int kPast = kH;          // floats k_mlp_backprop may read past the parameters (and drops)
constexpr int kStep = 32;          // pairs of samples k_mlp_wgrad loads at once

typedef float f32x4v __attribute__((ext_vector_type(4)));
typedef float f32x16v __attribute__((ext_vector_type(16)));

inline int pad32(int M) { return (M + 31) / 32 * 32; }

// activations and errors of a chunk: rows of samples, padded to whole tiles (errors of
// padding samples and of columns past M are zero)
struct Acts {
    float *h1, *h2, *d1, *d2, *dy;   // [chunk][kH] four times, [chunk][pad32(M)]
};

// Weights of U tiles of 16 units for K terms, in the order gemm16 uses them: lane l holds unit l % 16 of each
// tile and the terms 16 j + 4 (l / 16) + i.  A layer's loads are all in flight at once, and the next layer's
// are started before this one's products: one tile of samples per workgroup leaves nothing else to hide them.
template <int K, int U> struct Weights {
    float w[U][K / 4];
    template <class F> __device__ void load(F at)
    {
        const int g = (threadIdx.x & 63) >> 4;
#pragma unroll
        for (int k = 0; k < K / 4; ++k)
#pragma unroll
            for (int u = 0; u < U; ++u) w[u][k] = at(16 * (k / 4) + 4 * g + k % 4, u);
    }
    // from rows of n <= K terms at row(u), for products with a transposed matrix: four terms a load, the lanes
    // being rows apart; terms past n are read (kPast floats past the last row at most) and set to zero
    template <class F> __device__ void load_rows(int n, F row)
    {
        const int g = (threadIdx.x & 63) >> 4;
#pragma unroll
        for (int j = 0; j < K / 16; ++j)
#pragma unroll
            for (int u = 0; u < U; ++u) {
                const int k = 16 * j + 4 * g;
                float4 x;   // rows of any length: no alignment past a float's
                __builtin_memcpy(&x, row(u) + k, 16);
                w[u][4 * j] = k < n ? x.x : 0.f;
                w[u][4 * j + 1] = k + 1 < n ? x.y : 0.f;
                w[u][4 * j + 2] = k + 2 < n ? x.z : 0.f;
                w[u][4 * j + 3] = k + 3 < n ? x.w : 0.f;
            }
    }
};

// acc[u] (16 samples x 16 units of tile u) += in (LDS rows of `ld`) times w; lane l receives samples
// 4 (l / 16) .. + 3 of unit l % 16
template <int K, int U>
__device__ inline void gemm16(const float *in, int ld, const Weights<K, U> &w, f32x4v (&acc)[U])
{
    const int l = threadIdx.x & 63;
    const float *a = in + (l & 15) * ld + 4 * (l >> 4);
#pragma unroll
    for (int j = 0; j < K / 16; ++j) {
        const float4 x = *reinterpret_cast<const float4 *>(a + 16 * j);
        const float v[4] = {x.x, x.y, x.z, x.w};
#pragma unroll
        for (int i = 0; i < 4; ++i)
#pragma unroll
            for (int u = 0; u < U; ++u)
                acc[u] = __builtin_amdgcn_mfma_f32_16x16x4f32(v[i], w.w[u][4 * j + i], acc[u], 0, 0, 0);
    }
}

__global__ __launch_bounds__(kNT, 1) void k_mlp_backprop(const float *__restrict__ prm, int M, int MP, int64_t n,
                                                      const float *__restrict__ X, const int *__restrict__ idx,
                                                      const float *__restrict__ T, float inv_n, Acts out, int add,
                                                      double *__restrict__ lpart)
{
    constexpr int LH = kH + 4, LX = kD + 4;   // padded LDS rows
    __shared__ __attribute__((aligned(16))) float xs[kGS * LX], h1[kGS * LH], h2[kGS * LH], dy[kGS * LH], dz[kGS * LH];
    __shared__ double lsum[kNT / 64];
    const Offs of = offsets(M);
    const float *W1 = prm + of.w1, *B1 = prm + of.b1, *W2 = prm + of.w2, *B2 = prm + of.b2, *W3 = prm + of.w3,
                *B3 = prm + of.b3;
    const int t = threadIdx.x, w = t >> 6, l = t & 63, m = l & 15, g = l >> 4;
    double lacc = 0.0;
    const int64_t s0 = (int64_t)blockIdx.x * kGS;
    const int cnt = (int)min((int64_t)kGS, n - s0);
    for (int e = t; e < kGS * kD; e += kNT) {
        const int s = e / kD, k = e % kD;
        float v = 0.f;
        if (s < cnt) v = X[(idx ? (int64_t)idx[s0 + s] : s0 + s) * kD + k];
        xs[s * LX + k] = v;
    }
    // units of this wave: two tiles of a hidden layer, up to two of the outputs
    const int o0 = 32 * w + m, y0 = 16 * w + m;
    const bool in3[2] = {y0 < M, y0 + 64 < M};
    float c1[2], c2[2], c3[2], target[2][4];
    int64_t row[4];
#pragma unroll
    for (int i = 0; i < 4; ++i) {
        const int64_t s = s0 + min(4 * g + i, cnt - 1);
        row[i] = (idx ? (int64_t)idx[s] : s) * M;
    }
#pragma unroll
    for (int u = 0; u < 2; ++u) {
        const int y = min(y0 + 64 * u, M - 1);   // units past M are dropped below
        c1[u] = B1[o0 + 16 * u];
        c2[u] = B2[o0 + 16 * u];
        c3[u] = B3[y];
#pragma unroll
        for (int i = 0; i < 4; ++i) target[u][i] = T[row[i] + y];
    }
    Weights<kD, 2> w1;
    Weights<kH, 2> w2;
    w1.load([&](int k, int u) { return W1[k * kH + o0 + 16 * u]; });
    w2.load([&](int k, int u) { return W2[k * kH + o0 + 16 * u]; });
    __syncthreads();
    {   // h1 = tanh(x W1 + b1)
        f32x4v a[2] = {{c1[0], c1[0], c1[0], c1[0]}, {c1[1], c1[1], c1[1], c1[1]}};
        gemm16(xs, LX, w1, a);
#pragma unroll
        for (int u = 0; u < 2; ++u)
#pragma unroll
            for (int i = 0; i < 4; ++i) {
                const float h = tanhf(a[u][i]);
                h1[(4 * g + i) * LH + o0 + 16 * u] = h;
                out.h1[(s0 + 4 * g + i) * kH + o0 + 16 * u] = h;
            }
    }
    Weights<kH, 2> w3;
    w3.load([&](int k, int u) {   // units past M: some other weight, set to zero
        const float v = W3[k * M + y0 + 64 * u];
        return in3[u] ? v : 0.f;
    });
    __syncthreads();
    {   // h2 = tanh(h1 W2 + b2)
        f32x4v a[2] = {{c2[0], c2[0], c2[0], c2[0]}, {c2[1], c2[1], c2[1], c2[1]}};
        gemm16(h1, LH, w2, a);
#pragma unroll
        for (int u = 0; u < 2; ++u)
#pragma unroll
            for (int i = 0; i < 4; ++i) {
                const float h = tanhf(a[u][i]);
                h2[(4 * g + i) * LH + o0 + 16 * u] = h;
                out.h2[(s0 + 4 * g + i) * kH + o0 + 16 * u] = h;
            }
    }
    Weights<kH, 2> w3t;   // terms past M meet zero weights
    w3t.load_rows(M, [&](int u) { return W3 + (o0 + 16 * u) * M; });
    __syncthreads();
    {   // y = h2 W3 + b3, dy = (y - t) / n
        f32x4v a[2] = {{c3[0], c3[0], c3[0], c3[0]}, {c3[1], c3[1], c3[1], c3[1]}};
        gemm16(h2, LH, w3, a);
#pragma unroll
        for (int u = 0; u < 2; ++u) {
            const int o = y0 + 64 * u;
#pragma unroll
            for (int i = 0; i < 4; ++i) {
                const int s = 4 * g + i;
                float r = 0.f;
                if (in3[u] && s < cnt) r = a[u][i] - target[u][i];
                lacc += (double)(r * r);
                r *= inv_n;
                dy[s * LH + o] = r;
                if (o < MP) out.dy[(s0 + s) * MP + o] = r;
            }
        }
    }
    Weights<kH, 2> w2t;
    w2t.load_rows(kH, [&](int u) { return W2 + (o0 + 16 * u) * kH; });
    __syncthreads();
    {   // d2 = (dy W3^T) (1 - h2^2)
        f32x4v a[2] = {{0.f, 0.f, 0.f, 0.f}, {0.f, 0.f, 0.f, 0.f}};
        gemm16(dy, LH, w3t, a);
#pragma unroll
        for (int u = 0; u < 2; ++u)
#pragma unroll
            for (int i = 0; i < 4; ++i) {
                const int at = (4 * g + i) * LH + o0 + 16 * u;
                const float h = h2[at], d = a[u][i] * (1.f - h * h);
                dz[at] = d;
                out.d2[(s0 + 4 * g + i) * kH + o0 + 16 * u] = d;
            }
    }
    __syncthreads();
    {   // d1 = (d2 W2^T) (1 - h1^2)
        f32x4v a[2] = {{0.f, 0.f, 0.f, 0.f}, {0.f, 0.f, 0.f, 0.f}};
        gemm16(dz, LH, w2t, a);
#pragma unroll
        for (int u = 0; u < 2; ++u)
#pragma unroll
            for (int i = 0; i < 4; ++i) {
                const float h = h1[(4 * g + i) * LH + o0 + 16 * u];
                out.d1[(s0 + 4 * g + i) * kH + o0 + 16 * u] = a[u][i] * (1.f - h * h);
            }
    }
    lacc = wave_sum(lacc);
    if (l == 0) lsum[w] = lacc;
    __syncthreads();
    if (t == 0) {
        double s = add ? lpart[blockIdx.x] : 0.0;
        for (int q = 0; q < kNT / 64; ++q) s += lsum[q];
        lpart[blockIdx.x] = s;
    }
}

// One wave per 32 x 32 tile of a weight matrix and range of samples: part[range][...] (+)= in^T err over the
// range.  Tiles: 16 of W2, then 4 per 32 columns of W3, then 4 of W1; the tiles of the first input rows also
// sum the errors' columns, the bias gradients.
__global__ __launch_bounds__(64, 1) void k_mlp_wgrad(int M, int MP, int64_t n, const float *__restrict__ X,
                                                  const int *__restrict__ idx, Acts in, int add,
                                                  float *__restrict__ part)
{
    const Offs of = offsets(M);
    const int l = threadIdx.x, c = l & 31, kk = l >> 5, n3 = MP / 32;
    const int tile = blockIdx.x;
    const int64_t np = (n + kGS - 1) / kGS * kGS;   // padded samples
    const int64_t span = (np + gridDim.y * 2 - 1) / (gridDim.y * 2) * 2;
    const int64_t lo = min(np, span * blockIdx.y), hi = min(np, lo + span);
    float *out = part + of.total * blockIdx.y;
    const float *A, *E;
    int lda, lde, mt, nt, N, ldo;
    int64_t wo, bo;
    bool gather = false;
    if (tile < 16) {
        A = in.h1; lda = kH; E = in.d2; lde = kH; mt = tile >> 2; nt = tile & 3; N = kH; ldo = kH; wo = of.w2; bo = of.b2;
    } else if (tile < 16 + 4 * n3) {
        const int x = tile - 16;
        A = in.h2; lda = kH; E = in.dy; lde = MP; mt = x / n3; nt = x % n3; N = M; ldo = M; wo = of.w3; bo = of.b3;
    } else {
        A = X; lda = kD; E = in.d1; lde = kH; mt = 0; nt = tile - 16 - 4 * n3; N = kH; ldo = kH; wo = of.w1; bo = of.b1;
        gather = true;
    }
    const float *e = E + 32 * nt + c;
    f32x16v acc;
#pragma unroll
    for (int i = 0; i < 16; ++i) acc[i] = 0.f;
    float bias = 0.f;
    const float *a = A + 32 * mt + c;
    for (int64_t s0 = lo; s0 < hi; s0 += 2 * kStep) {
        float x[kStep], d[kStep];   // all loads of a step in flight; zeros past the range
#pragma unroll
        for (int u = 0; u < kStep; ++u) {
            const int64_t r = s0 + 2 * u + kk;
            const bool live = r < hi && (!gather || r < n);
            const int64_t q = live ? r : 0, row = gather && idx ? (int64_t)idx[q] : q;
            x[u] = a[row * lda];
            d[u] = e[q * lde];
            if (!live) x[u] = d[u] = 0.f;
        }
#pragma unroll
        for (int u = 0; u < kStep; ++u) {
            bias += d[u];
            acc = __builtin_amdgcn_mfma_f32_32x32x2f32(x[u], d[u], acc, 0, 0, 0);
        }
    }
    const int o = 32 * nt + c;
    if (o < N) {
#pragma unroll
        for (int i = 0; i < 16; ++i) {
            const int r = 32 * mt + 8 * (i >> 2) + 4 * kk + (i & 3);
            const int64_t at = wo + (int64_t)r * ldo + o;
            out[at] = add ? out[at] + acc[i] : acc[i];
        }
    }
    bias += __shfl_xor(bias, 32, 64);
    if (mt == 0 && kk == 0 && o < N) out[bo + o] = add ? out[bo + o] + bias : bias;
}

// grad[p] = sum over parts w (ascending) of part[w][p]; the last workgroup: loss[0] (+)= scale * sum of the
// loss parts, in a fixed tree.
__global__ __launch_bounds__(256) void k_sum_gradient(int64_t P, int parts, const float *__restrict__ part,
                                                      float *__restrict__ grad, int lparts,
                                                      const double *__restrict__ lpart, double scale, int accumulate,
                                                      double *__restrict__ loss)
{
    __shared__ double red[256];
    if (blockIdx.x == gridDim.x - 1) {
        double s = 0.0;
        for (int w = threadIdx.x; w < lparts; w += 256) s += lpart[w];
        red[threadIdx.x] = s;
        __syncthreads();
        for (int off = 128; off > 0; off >>= 1) {
            if ((int)threadIdx.x < off) red[threadIdx.x] += red[threadIdx.x + off];
            __syncthreads();
        }
        if (threadIdx.x == 0) loss[0] = (accumulate ? loss[0] : 0.0) + scale * red[0];
        return;
    }
    const int64_t p = (int64_t)blockIdx.x * 256 + threadIdx.x;
    if (p >= P) return;
    float s = 0.f;
#pragma unroll 8
    for (int w = 0; w < parts; ++w) s += part[(int64_t)w * P + p];
    grad[p] = s;
}

__global__ void k_adam(int64_t P, float *__restrict__ prm, float *__restrict__ m, float *__restrict__ v,
                       const float *__restrict__ g, float lr, float b1, float b2, float eps, float c1, float c2)
{
    const int64_t p = (int64_t)blockIdx.x * blockDim.x + threadIdx.x;
    if (p >= P) return;
    const float gp = g[p];
    const float mp = b1 * m[p] + (1.f - b1) * gp;
    const float vp = b2 * v[p] + (1.f - b2) * gp * gp;
    m[p] = mp;
    v[p] = vp;
    prm[p] -= lr * (mp * c1) / (sqrtf(vp * c2) + eps);
}

// ------------------------------------------------------------------ BF16 inference

typedef short bf16x4 __attribute__((ext_vector_type(4)));
typedef float f32x4 __attribute__((ext_vector_type(4)));

// round to nearest even; NaN stays NaN, infinities stay infinite (one instruction for two)
__device__ inline unsigned short bf16_bits(float f) { return __builtin_bit_cast(unsigned short, (__bf16)f); }

// Pack a K x N input-major weight matrix into the B-operand layout of the
// 16x16x16 BF16 MFMA: tile (kt, nt), lane l, element e holds
// W[16 kt + 4 (l / 16) + e][16 nt + l % 16] (zero outside the matrix).
__global__ void k_pack_bf16(const float *__restrict__ W, int K, int N, int KT, int NTl, unsigned short *__restrict__ out)
{
    const int64_t q = (int64_t)blockIdx.x * blockDim.x + threadIdx.x;
    if (q >= (int64_t)KT * NTl * 256) return;
    const int e = (int)(q & 3), l = (int)((q >> 2) & 63);
    const int nt = (int)((q >> 8) % NTl), kt = (int)((q >> 8) / NTl);
    const int k = 16 * kt + 4 * (l >> 4) + e, c = 16 * nt + (l & 15);
    out[q] = (k < K && c < N) ? bf16_bits(W[(int64_t)k * N + c]) : (unsigned short)0;
}

constexpr int kKT1 = kD / 16;        // k-steps of the first layer
constexpr int kBW = 16;              // wavefronts of a workgroup
constexpr int kBGrid = 256;          // workgroups, at most: one per CU

__device__ inline bf16x4 bf16_of(const f32x4 &v)
{
    bf16x4 r;
#pragma unroll
    for (int e = 0; e < 4; ++e) r[e] = (short)bf16_bits(v[e]);
    return r;
}

// acc[nt] = sum over kt of weights(kt, nt)^T act[kt], units by samples
template <int KT, int NTl> __device__ inline void layer(const bf16x4 *p, const bf16x4 *act, f32x4 (&acc)[NTl])
{
    const int l = threadIdx.x & 63;
#pragma unroll
    for (int nt = 0; nt < NTl; ++nt) acc[nt] = f32x4{0.f, 0.f, 0.f, 0.f};
#pragma unroll
    for (int kt = 0; kt < KT; ++kt)
#pragma unroll
        for (int nt = 0; nt < NTl; ++nt)
            acc[nt] = __builtin_amdgcn_mfma_f32_16x16x16bf16_1k(p[(kt * NTl + nt) * 64 + l], act[kt], acc[nt], 0, 0, 0);
}

// One wavefront per tile of 16 samples, tiles in turn.  The layers are computed transposed, units by samples:
// lane l receives units 4 (l / 16) .. + 3 of sample l % 16 of each 16 x 16 result, which after the tanh are
// exactly the four terms it supplies to the next layer's products, so activations never leave the registers.
// The weights of all layers (64 KB at 81 outputs) stay in LDS for all of a workgroup's tiles; a tile's outputs,
// contiguous in memory, are turned through 8 rows of LDS into whole lines.  What bounds it is the vector work
// of 256 tanh and roundings a sample.  The former kernel read every weight from memory per 16 samples into 340
// registers, one wavefront per SIMD with little in flight, and kept activations in LDS: 1828 us for the 856
// thousand blocks of 4096 atoms at 10 A, b = 9; this one 239 us.
template <int NT3>
__global__ __launch_bounds__(64 * kBW) void k_mlp_bf16(const unsigned short *__restrict__ P1,
                                                       const unsigned short *__restrict__ P2,
                                                       const unsigned short *__restrict__ P3,
                                                       const float *__restrict__ B1, const float *__restrict__ B2,
                                                       const float *__restrict__ B3, int M, int64_t n,
                                                       const float *__restrict__ X, Out out)
{
    constexpr int N1 = kKT1 * 8 * 64, N2 = 8 * 8 * 64, N3 = 8 * NT3 * 64;   // fragments of four
    __shared__ bf16x4 p[N1 + N2 + N3];
    __shared__ __attribute__((aligned(16))) float bias[3 * kH];
    __shared__ float stage[kBW][8 * 16 * NT3];
    const int t = threadIdx.x, w = t >> 6, l = t & 63, m = l & 15, kq = l >> 4;
    for (int e = t; e < N1; e += 64 * kBW) p[e] = reinterpret_cast<const bf16x4 *>(P1)[e];
    for (int e = t; e < N2; e += 64 * kBW) p[N1 + e] = reinterpret_cast<const bf16x4 *>(P2)[e];
    for (int e = t; e < N3; e += 64 * kBW) p[N1 + N2 + e] = reinterpret_cast<const bf16x4 *>(P3)[e];
    if (t < kH) {
        bias[t] = B1[t];
        bias[kH + t] = B2[t];
        bias[2 * kH + t] = t < M ? B3[t] : 0.f;
    }
    __syncthreads();
    const int64_t tiles = (n + 15) / 16, step = (int64_t)gridDim.x * kBW;
    float *st = stage[w];
    // wavefronts of different workgroups take neighbouring tiles, so that few tiles fill the chip
    int64_t tile = blockIdx.x + (int64_t)w * gridDim.x;
    f32x4 x[kKT1];
    const auto fetch = [&](int64_t at) {
#pragma unroll
        for (int kt = 0; kt < kKT1; ++kt) {
            x[kt] = f32x4{0.f, 0.f, 0.f, 0.f};
            if (at * 16 + m < n) x[kt] = *reinterpret_cast<const f32x4 *>(X + (at * 16 + m) * kD + kt * 16 + 4 * kq);
        }
    };
    if (tile < tiles) fetch(tile);
    for (; tile < tiles; tile += step) {
        bf16x4 a[8];
#pragma unroll
        for (int kt = 0; kt < kKT1; ++kt) a[kt] = bf16_of(x[kt]);
        if (tile + step < tiles) fetch(tile + step);   // the next tile's inputs
        f32x4 acc[8];
        const auto activate = [&](const float *b) {
#pragma unroll
            for (int nt = 0; nt < 8; ++nt) {
                const f32x4 c = *reinterpret_cast<const f32x4 *>(b + nt * 16 + 4 * kq);
#pragma unroll
                for (int e = 0; e < 4; ++e) acc[nt][e] = tanhf(acc[nt][e] + c[e]);
                a[nt] = bf16_of(acc[nt]);
            }
        };
        layer<kKT1, 8>(p, a, acc);
        activate(bias);
        layer<8, 8>(p + N1, a, acc);
        activate(bias + kH);
        f32x4 y[NT3];
        layer<8, NT3>(p + N1 + N2, a, y);
#pragma unroll
        for (int half = 0; half < 2; ++half) {
            const int64_t s0 = tile * 16 + 8 * half;
            wave_sync();   // the rows before have been read
            if (m >> 3 == half)
#pragma unroll
                for (int nt = 0; nt < NT3; ++nt)
#pragma unroll
                    for (int e = 0; e < 4; ++e) {
                        const int col = nt * 16 + 4 * kq + e;
                        if (col < M) st[(m & 7) * M + col] = y[nt][e] + bias[2 * kH + col];
                    }
            wave_sync();
            const int cnt = (int)max((int64_t)0, min((int64_t)8, n - s0)) * M;
            for (int e = l; e < cnt; e += 64) put(out, s0 * M + e, st[e]);
        }
    }
}

using Bf16Kernel = void (*)(const unsigned short *, const unsigned short *, const unsigned short *, const float *,
                            const float *, const float *, int, int64_t, const float *, Out);
// by the tiles of 16 outputs
constexpr Bf16Kernel kMlpBf16[8] = {k_mlp_bf16<1>, k_mlp_bf16<2>, k_mlp_bf16<3>, k_mlp_bf16<4>,
                                    k_mlp_bf16<5>, k_mlp_bf16<6>, k_mlp_bf16<7>, k_mlp_bf16<8>};

__global__ void k_fill_f64(int64_t n, double v, double *__restrict__ x)
{
    const int64_t i = (int64_t)blockIdx.x * blockDim.x + threadIdx.x;
    if (i < n) x[i] = v;
}

__global__ void k_targets(int64_t n, const double *__restrict__ A, const double *__restrict__ B, double scale,
                          float *__restrict__ T)
{
    const int64_t i = (int64_t)blockIdx.x * blockDim.x + threadIdx.x;
    if (i < n) T[i] = (float)((A[i] - B[i]) / scale);
}

unsigned grid_for(int64_t n, int bs) { return (unsigned)((n + bs - 1) / bs); }

}  // namespace
}  // namespace bsm

using namespace bsm;

struct bsm_mlp_s {
    Context *c = nullptr;
    int M = 0;
    int64_t P = 0;
    DevBuf prm, m, v, grad, work, lpart, loss, pk1, pk2, pk3;   // work: activations, then partial gradients
    bool packed = false;
    int64_t t = 0;   // Adam steps taken

    int nt3() const { return (M + 15) / 16; }

    void pack()
    {
        if (packed) return;
        const Offs of = offsets(M);
        hipStream_t st = c->stream;
        const float *p = prm.as<float>();
        k_pack_bf16<<<grid_for(kKT1 * 8 * 256, 256), 256, 0, st>>>(p + of.w1, kD, kH, kKT1, 8, pk1.as<unsigned short>());
        k_pack_bf16<<<grid_for(8 * 8 * 256, 256), 256, 0, st>>>(p + of.w2, kH, kH, 8, 8, pk2.as<unsigned short>());
        k_pack_bf16<<<grid_for((int64_t)8 * nt3() * 256, 256), 256, 0, st>>>(p + of.w3, kH, M, 8, nt3(),
                                                                            pk3.as<unsigned short>());
        BSM_HIP_TRY(hipGetLastError());
        packed = true;
    }

    void forward(int precision, int64_t n, const float *X, const Out &out)
    {
        BSM_REQUIRE(precision == BSM_F32 || precision == BSM_BF16, BSM_EINVAL, "precision must be BSM_F32 or BSM_BF16");
        if (n == 0) return;
        BSM_REQUIRE(reinterpret_cast<uintptr_t>(X) % 16 == 0, BSM_EINVAL, "X must be 16-byte aligned");
        hipStream_t st = c->stream;
        if (precision == BSM_F32) {
            const int64_t tiles = (n + kTS - 1) / kTS;
            const unsigned grid = (unsigned)std::min<int64_t>(tiles, 4096);
            k_mlp_f32<<<grid, kNT, 0, st>>>(prm.as<float>(), M, n, X, out);
        } else {
            pack();
            const Offs of = offsets(M);
            const float *p = prm.as<float>();
            const unsigned grid = (unsigned)std::min<int64_t>((n + 15) / 16, kBGrid);
            kMlpBf16[nt3() - 1]<<<grid, 64 * kBW, 0, st>>>(pk1.as<unsigned short>(), pk2.as<unsigned short>(),
                                                           pk3.as<unsigned short>(), p + of.b1, p + of.b2, p + of.b3, M,
                                                           n, X, out);
        }
        BSM_HIP_TRY(hipGetLastError());
    }

    // gradient of the minibatch (n samples; rows idx[s] or s) into g; the loss sum (times `scale`)
    // into *loss_out (device-visible), added when `accumulate`
    void loss_grad(int64_t n, const float *X, const int *idx, const float *T, double scale, int accumulate, float *g,
                   double *loss_out)
    {
        hipStream_t st = c->stream;
        const int MP = pad32(M);
        float *x = work.as<float>(), *gpart = x + (int64_t)kGradChunk * (4 * kH + MP);
        const Acts a{x, x + (int64_t)kGradChunk * kH, x + (int64_t)kGradChunk * 2 * kH, x + (int64_t)kGradChunk * 3 * kH,
                     x + (int64_t)kGradChunk * 4 * kH};
        int splits = 0, lparts = 0;
        for (int64_t s0 = 0; s0 < n; s0 += kGradChunk) {
            const int64_t cnt = std::min<int64_t>(kGradChunk, n - s0);
            const int64_t tiles = (cnt + kGS - 1) / kGS;
            // a first chunk is the largest: later ones leave its other parts as they are
            if (s0 == 0) {
                splits = (int)std::min<int64_t>(kSplits, (tiles + 3) / 4);
                lparts = (int)tiles;
            }
            const float *Xc = idx ? X : X + s0 * kD, *Tc = idx ? T : T + s0 * M;
            const int *ic = idx ? idx + s0 : nullptr;
            k_mlp_backprop<<<(unsigned)tiles, kNT, 0, st>>>(prm.as<float>(), M, MP, cnt, Xc, ic, Tc, (float)(1.0 / (double)n), a,
                                                 s0 > 0, lpart.as<double>());
            k_mlp_wgrad<<<dim3(16 + 4 * (MP / 32) + 4, splits), 64, 0, st>>>(M, MP, cnt, Xc, ic, a, s0 > 0,
                                                                             gpart);
        }
        k_sum_gradient<<<grid_for(P, 256) + 1, 256, 0, st>>>(P, splits, gpart, g, lparts,
                                                             lpart.as<double>(), scale, accumulate, loss_out);
        BSM_HIP_TRY(hipGetLastError());
    }

    void adam(const bsm_adam &o, const float *g)
    {
        BSM_REQUIRE(o.lr > 0.f && o.beta1 >= 0.f && o.beta1 < 1.f && o.beta2 >= 0.f && o.beta2 < 1.f && o.eps >= 0.f,
                    BSM_EINVAL, "bad Adam parameters");
        ++t;
        const double c1 = 1.0 / (1.0 - std::pow((double)o.beta1, (double)t));
        const double c2 = 1.0 / (1.0 - std::pow((double)o.beta2, (double)t));
        k_adam<<<grid_for(P, 256), 256, 0, c->stream>>>(P, prm.as<float>(), m.as<float>(), v.as<float>(), g, o.lr,
                                                        o.beta1, o.beta2, o.eps, (float)c1, (float)c2);
        BSM_HIP_TRY(hipGetLastError());
        packed = false;
    }

    void clear_adam()
    {
        hipStream_t st = c->stream;
        BSM_HIP_TRY(hipMemsetAsync(m.ptr, 0, sizeof(float) * P, st));
        BSM_HIP_TRY(hipMemsetAsync(v.ptr, 0, sizeof(float) * P, st));
        t = 0;
    }
};

#define MLP_TRY try {
#define MLP_CATCH                                                  \
    }                                                              \
    catch (const Error &e) { return fail(e.code, e.msg); }         \
    catch (...) { return fail(BSM_EINVAL, "unknown error"); }

extern "C" {

int64_t bsm_mlp_param_count(const bsm_mlp_shape *shape)
{
    if (!shape || shape->width != kH || shape->out_dim < 1 || shape->out_dim > kH) return BSM_EINVAL;
    return offsets(shape->out_dim).total;
}

int bsm_mlp_create(bsm_ctx ctx, const bsm_mlp_shape *shape, const float *params, bsm_mlp *out)
{
    MLP_TRY
    BSM_REQUIRE(ctx && shape && params && out, BSM_EINVAL, "NULL argument");
    BSM_REQUIRE(shape->width == kH, BSM_EINVAL, "hidden width must be 128");
    BSM_REQUIRE(shape->out_dim >= 1 && shape->out_dim <= kH, BSM_EINVAL, "out_dim must be 1..128");
    std::unique_ptr<bsm_mlp_s> net(new bsm_mlp_s());
    Context *c = &ctx->c;
    net->c = c;
    net->M = shape->out_dim;
    net->P = offsets(net->M).total;
    const size_t pb = sizeof(float) * (size_t)net->P;
    net->prm = DevBuf(c, pb + sizeof(float) * kPast);
    net->m = DevBuf(c, pb);
    net->v = DevBuf(c, pb);
    net->grad = DevBuf(c, pb);
    net->work = DevBuf(c, sizeof(float) * (size_t)kGradChunk * (4 * kH + pad32(net->M)) + pb * kSplits);
    net->lpart = DevBuf(c, sizeof(double) * (kGradChunk / kGS));
    net->loss = DevBuf(c, sizeof(double) * 2);
    net->pk1 = DevBuf(c, sizeof(unsigned short) * kKT1 * 8 * 256);
    net->pk2 = DevBuf(c, sizeof(unsigned short) * 8 * 8 * 256);
    net->pk3 = DevBuf(c, sizeof(unsigned short) * 8 * (size_t)net->nt3() * 256);
    BSM_HIP_TRY(hipMemcpyAsync(net->prm.ptr, params, pb, hipMemcpyHostToDevice, c->stream));
    net->clear_adam();
    BSM_HIP_TRY(hipStreamSynchronize(c->stream));
    *out = net.release();
    return BSM_OK;
    MLP_CATCH
}

int bsm_mlp_get_params(bsm_mlp net, float *params)
{
    MLP_TRY
    BSM_REQUIRE(net && params, BSM_EINVAL, "NULL argument");
    BSM_HIP_TRY(hipMemcpyAsync(params, net->prm.ptr, sizeof(float) * net->P, hipMemcpyDeviceToHost, net->c->stream));
    BSM_HIP_TRY(hipStreamSynchronize(net->c->stream));
    return BSM_OK;
    MLP_CATCH
}

int bsm_mlp_set_params(bsm_mlp net, const float *params)
{
    MLP_TRY
    BSM_REQUIRE(net && params, BSM_EINVAL, "NULL argument");
    BSM_HIP_TRY(hipMemcpyAsync(net->prm.ptr, params, sizeof(float) * net->P, hipMemcpyHostToDevice, net->c->stream));
    net->clear_adam();
    net->packed = false;
    BSM_HIP_TRY(hipStreamSynchronize(net->c->stream));
    return BSM_OK;
    MLP_CATCH
}

int bsm_mlp_destroy(bsm_mlp net)
{
    if (net) {
        (void)hipStreamSynchronize(net->c->stream);
        delete net;
    }
    return BSM_OK;
}

int bsm_pair_descriptors(bsm_ctx ctx, bsm_pattern NP, bsm_pattern P, float *desc)
{
    MLP_TRY
    BSM_REQUIRE(ctx && NP && P && desc, BSM_EINVAL, "NULL argument");
    BSM_REQUIRE(reinterpret_cast<uintptr_t>(desc) % 16 == 0, BSM_EINVAL, "desc must be 16-byte aligned");
    BSM_REQUIRE(NP->natoms == P->natoms && NP->box[0] == P->box[0] && NP->box[1] == P->box[1] &&
                    NP->box[2] == P->box[2],
                BSM_EPATTERN, "neighbour pattern is over other atoms");
    Context *c = &ctx->c;
    hipStream_t st = c->stream;
    const int n = P->natoms;
    const double3 box = make_double3(P->box[0], P->box[1], P->box[2]);
    DevBuf fr(c, sizeof(double) * kFrame * (size_t)std::max(1, n)), bad(c, sizeof(int));
    BSM_HIP_TRY(hipMemsetAsync(bad.ptr, 0, sizeof(int), st));
    k_atom_frames<<<grid_for(n, kFrameAtoms), kFrameAtoms * kFrameLanes, 0, st>>>(n, NP->pos.as<double>(), box, NP->rowptr.as<int>(),
                                                    NP->cols.as<int>(), fr.as<double>(), bad.as<int>());
    BSM_HIP_TRY(hipGetLastError());
    int hbad = 0;
    BSM_HIP_TRY(hipMemcpyAsync(&hbad, bad.ptr, sizeof(int), hipMemcpyDeviceToHost, st));
    BSM_HIP_TRY(hipStreamSynchronize(st));
    BSM_REQUIRE(!hbad, BSM_EINVAL, "an atom has fewer than four neighbours in the neighbour pattern");
    if (P->nnzb > 0)
        k_pair_desc<<<grid_for(P->nnzb, kDescSlots), kDescSlots, 0, st>>>(P->nnzb, P->rowidx.as<int>(), P->cols.as<int>(),
                                                            P->pos.as<double>(), box, P->cutoff, fr.as<double>(),
                                                            desc);
    BSM_HIP_TRY(hipGetLastError());
    BSM_HIP_TRY(hipStreamSynchronize(st));   // the frames buffer is released on return
    return BSM_OK;
    MLP_CATCH
}

int bsm_mlp_forward(bsm_mlp net, int precision, int64_t n, const float *X, float *Y)
{
    MLP_TRY
    BSM_REQUIRE(net && n >= 0 && (n == 0 || (X && Y)), BSM_EINVAL, "bad argument");
    net->forward(precision, n, X, Out{Y, nullptr, 0.0, 0.0});
    return BSM_OK;
    MLP_CATCH
}

int bsm_mlp_loss_grad(bsm_mlp net, int64_t n, const float *X, const float *T, double *loss, float *grad)
{
    MLP_TRY
    BSM_REQUIRE(net && X && T && grad && n >= 1, BSM_EINVAL, "bad argument");
    double *host = net->c->host_scalars;   // pinned
    net->loss_grad(n, X, nullptr, T, 0.5 / (double)n, 0, grad, host);
    BSM_HIP_TRY(hipStreamSynchronize(net->c->stream));
    if (loss) *loss = *host;
    return BSM_OK;
    MLP_CATCH
}

int bsm_mlp_adam_step(bsm_mlp net, const bsm_adam *opt, const float *grad)
{
    MLP_TRY
    BSM_REQUIRE(net && opt && grad, BSM_EINVAL, "NULL argument");
    net->adam(*opt, grad);
    return BSM_OK;
    MLP_CATCH
}

int bsm_mlp_train(bsm_mlp net, const bsm_mlp_train_params *p, int64_t n, const float *X, const float *T,
                  const int32_t *perm, double *epoch_loss)
{
    MLP_TRY
    BSM_REQUIRE(net && p && X && T && n >= 1, BSM_EINVAL, "bad argument");
    BSM_REQUIRE(p->epochs >= 0 && p->batch >= 1, BSM_EINVAL, "bad epochs or batch");
    hipStream_t st = net->c->stream;
    const int64_t nb = (n + p->batch - 1) / p->batch;
    for (int e = 0; e < p->epochs; ++e) {
        for (int64_t k = 0; k < nb; ++k) {
            const int64_t s0 = k * p->batch, cnt = std::min<int64_t>(p->batch, n - s0);
            const double scale = 0.5 / (double)cnt / (double)nb;   // mean over minibatches
            if (perm)
                net->loss_grad(cnt, X, perm + s0, T, scale, k > 0, net->grad.as<float>(), net->loss.as<double>());
            else
                net->loss_grad(cnt, X + s0 * kD, nullptr, T + s0 * net->M, scale, k > 0, net->grad.as<float>(),
                               net->loss.as<double>());
            net->adam(p->opt, net->grad.as<float>());
        }
        double h = 0.0;
        BSM_HIP_TRY(hipMemcpyAsync(&h, net->loss.ptr, sizeof(double), hipMemcpyDeviceToHost, st));
        BSM_HIP_TRY(hipStreamSynchronize(st));
        if (epoch_loss) epoch_loss[e] = h;
    }
    return BSM_OK;
    MLP_CATCH
}

int bsm_mlp_targets(bsm_ctx ctx, const bsm_matrix *A, const bsm_matrix *B, double scale, float *T)
{
    MLP_TRY
    BSM_REQUIRE(ctx && T, BSM_EINVAL, "NULL argument");
    check_matrix(A, "A");
    check_matrix(B, "B");
    BSM_REQUIRE(A->pattern == B->pattern, BSM_EPATTERN, "A and B must share a pattern");
    BSM_REQUIRE(scale != 0.0 && std::isfinite(scale), BSM_EINVAL, "scale must be finite and non-zero");
    const int64_t ne = nelems(A->pattern);
    if (ne > 0)
        k_targets<<<grid_for(ne, 256), 256, 0, ctx->c.stream>>>(ne, (const double *)A->blocks,
                                                              (const double *)B->blocks, scale, T);
    BSM_HIP_TRY(hipGetLastError());
    return BSM_OK;
    MLP_CATCH
}

int bsm_mlp_predict_blocks(bsm_mlp net, int precision, const float *X, double scale, double beta,
                           const bsm_matrix *M)
{
    MLP_TRY
    BSM_REQUIRE(net && X, BSM_EINVAL, "NULL argument");
    check_matrix(M, "M");
    const int b = M->pattern->b;
    BSM_REQUIRE(b * b == net->M, BSM_EPATTERN, "network out_dim must be b^2");
    net->forward(precision, M->pattern->nnzb, X, Out{nullptr, (double *)M->blocks, scale, beta});
    return BSM_OK;
    MLP_CATCH
}

}  // extern "C"
