// Pattern-local elementwise kernels: axpby, blockwise symmetrisation and
// transposition, masked copies between patterns, identity and block input.
// All are HBM-bound streams over the block arrays.
#include "bsm_internal.h"

namespace bsm {
namespace {

constexpr int kT = 256;

inline unsigned grid1(int64_t n) { return (unsigned)std::max<int64_t>(1, (n + kT - 1) / kT); }

__global__ void k_axpby(int64_t n, double a, const double *x, double b, double *y)
{
    int64_t e = (int64_t)blockIdx.x * kT + threadIdx.x;
    if (e >= n) return;
    if (b == 0.0) {
        y[e] = a * x[e];
        return;
    }
    const double xv = x[e], yv = y[e];   // both loads under one wait
    y[e] = fma(b, yv, a * xv);
}

// The same for 16-byte aligned arrays of an even count, a pair per thread (each element is the fma
// above, written out so that both give the same bits).
__global__ __launch_bounds__(kT) void k_axpby2(int64_t n2, double a, const double2 *x, double b, double2 *y)
{
    const int64_t e = (int64_t)blockIdx.x * kT + threadIdx.x;
    if (e >= n2) return;
    const double2 xv = x[e];
    double2 v = make_double2(a * xv.x, a * xv.y);
    if (b != 0.0) {
        const double2 yv = y[e];
        v = make_double2(fma(b, yv.x, v.x), fma(b, yv.y, v.y));
    }
    y[e] = v;
}

// z <- a x + b y + c z, one element per thread (x or y may be z).  Each element
// is fma(c, z, fma(a, x, b y)), written out so that the paired kernel below
// gives the same bits.
__global__ void k_axpbypcz(int64_t n, double a, const double *x, double b, const double *y, double c,
                           double *z)
{
    int64_t e = (int64_t)blockIdx.x * kT + threadIdx.x;
    if (e >= n) return;
    const double v = fma(a, x[e], b * y[e]);
    z[e] = (c == 0.0) ? v : fma(c, z[e], v);
}

// The same for an even count of 16-byte aligned elements, a pair per thread.
__global__ __launch_bounds__(kT) void k_axpbypcz2(int64_t n2, double a, const double2 *x, double b, const double2 *y,
                                                  double c, double2 *z)
{
    const int64_t e = (int64_t)blockIdx.x * kT + threadIdx.x;
    if (e >= n2) return;
    const double2 xv = x[e], yv = y[e];
    double2 v = make_double2(fma(a, xv.x, b * yv.x), fma(a, xv.y, b * yv.y));
    if (c != 0.0) {
        const double2 zv = z[e];
        v = make_double2(fma(c, zv.x, v.x), fma(c, zv.y, v.y));
    }
    z[e] = v;
}

constexpr int kUnroll = 4;   // elements per thread of the kernels below

// In place (M_ij, M_ji) <- ((M_ij + M_ji^T)/2, its transpose).  The thread of
// element (p, q) of slot s with s < t (or s == t and p <= q) writes both partners.
// U elements per thread, all loads before the stores.
template <int BC, int U>
__global__ __launch_bounds__(kT) void k_symmetrize(int64_t nnz, int b_arg, const int *__restrict__ tmap, double *M)
{
    const int b = BC > 0 ? BC : b_arg, bb = b * b;
    const int64_t nel = nnz * bb, e0 = (int64_t)blockIdx.x * (kT * U) + threadIdx.x;
    int64_t at[U];
    double x[U], y[U];
#pragma unroll
    for (int u = 0; u < U; ++u) {
        const int64_t e = e0 + u * kT;
        at[u] = -1;
        if (e >= nel) continue;
        const int64_t s = e / bb;
        const int r = (int)(e - s * bb), p = r / b, q = r - p * b;
        const int64_t t = tmap[s];
        if (t < s || (t == s && p > q)) continue;
        at[u] = t * bb + q * b + p;
    }
#pragma unroll
    for (int u = 0; u < U; ++u)
        if (at[u] >= 0) {
            x[u] = M[e0 + u * kT];
            y[u] = M[at[u]];
        }
#pragma unroll
    for (int u = 0; u < U; ++u)
        if (at[u] >= 0) {
            const double v = 0.5 * (x[u] + y[u]);
            M[e0 + u * kT] = v;
            M[at[u]] = v;
        }
}

// L <- L + a D + delta P_N, then symmetrised in place as k_symmetrize does, in one pass; a, delta and
// whether to step at all come from device memory.
template <int BC>
__global__ __launch_bounds__(kT) void k_cg_update(int64_t nnz, int b_arg, const int *__restrict__ tmap,
                                                  const double *__restrict__ min, const double *__restrict__ D,
                                                  const double *__restrict__ PN, double *L)
{
    if (min[2] != 0.0) return;
    const double a = min[0], delta = min[1];
    const int b = BC > 0 ? BC : b_arg, bb = b * b;
    const int64_t nel = nnz * bb, e0 = (int64_t)blockIdx.x * (kT * kUnroll) + threadIdx.x;
    int64_t at[kUnroll];
    double x[kUnroll], y[kUnroll];
#pragma unroll
    for (int u = 0; u < kUnroll; ++u) {
        const int64_t e = e0 + u * kT;
        at[u] = -1;
        if (e >= nel) continue;
        const int64_t s = e / bb;
        const int r = (int)(e - s * bb), p = r / b, q = r - p * b;
        const int64_t t = tmap[s];
        if (t < s || (t == s && p > q)) continue;
        at[u] = t * bb + q * b + p;
    }
#pragma unroll
    for (int u = 0; u < kUnroll; ++u)
        if (at[u] >= 0) {
            const int64_t e = e0 + u * kT, f = at[u];
            x[u] = fma(1.0, L[e], fma(a, D[e], delta * PN[e]));
            y[u] = fma(1.0, L[f], fma(a, D[f], delta * PN[f]));
        }
#pragma unroll
    for (int u = 0; u < kUnroll; ++u)
        if (at[u] >= 0) {
            const double v = 0.5 * (x[u] + y[u]);
            L[e0 + u * kT] = v;
            L[at[u]] = v;
        }
}

// out[s] <- alpha (M[s] + M[t]^T) + beta out[s]
template <int BC>
__global__ void k_add_transpose(int64_t nnz, int b_arg, const int *__restrict__ tmap, double alpha,
                                const double *__restrict__ M, double beta, double *__restrict__ out)
{
    const int b = BC > 0 ? BC : b_arg, bb = b * b;
    int64_t e = (int64_t)blockIdx.x * kT + threadIdx.x;
    if (e >= nnz * bb) return;
    const int64_t s = e / bb;
    const int r = (int)(e - s * bb), p = r / b, q = r - p * b;
    const int64_t t = tmap[s];
    const double v = alpha * (M[e] + M[t * bb + q * b + p]);
    out[e] = (beta == 0.0) ? v : v + beta * out[e];
}

__device__ inline int find_in_row(const int *__restrict__ rowptr, const int *__restrict__ cols, int i, int j)
{
    int lo = rowptr[i], hi = rowptr[i + 1], end = hi;
    while (lo < hi) {
        int mid = (lo + hi) >> 1;
        if (cols[mid] < j) lo = mid + 1;
        else hi = mid;
    }
    return (lo < end && cols[lo] == j) ? lo : -1;
}

// One workgroup per chunk of destination slots: look up the source slot, copy or zero.
// A chunk has to be small where there are few of them, so that workgroups cover the loads (b = 9,
// onto 4096 atoms, 6 A: 26 us with 64 slots, 30 with 256; 216 atoms, 6.4 and 15.9), and large where
// they are many and their blocks small, as all the threads of a workgroup look a slot up and with 64
// slots three quarters idle meanwhile (b = 4, onto 4096 atoms, 10 A: 32.7 us with 64, 24.5 with 256;
// b = 1, 11.9 and 5.8; b = 9, 16 A, 790 and 677).
constexpr int kFewMaskSlots = 64, kManyMaskSlots = kT;
inline bool many_mask_slots(int64_t nnz, int b) { return nnz >= (b <= 5 ? 1 << 17 : 1 << 21); }
template <int BC, int kMaskSlots>
__global__ __launch_bounds__(kT) void k_mask_copy(int64_t nnzd, int b_arg, const int *__restrict__ rowsD,
                                                  const int *__restrict__ colsD, const int *__restrict__ rpS,
                                                  const int *__restrict__ colsS, const double *__restrict__ src,
                                                  double *__restrict__ dst)
{
    __shared__ int ss[kMaskSlots];
    const int b = BC > 0 ? BC : b_arg, bb = b * b;
    const int64_t base = (int64_t)blockIdx.x * kMaskSlots;
    const int nsl = (int)min((int64_t)kMaskSlots, nnzd - base);
    if (threadIdx.x < nsl) {
        const int64_t s = base + threadIdx.x;
        ss[threadIdx.x] = find_in_row(rpS, colsS, rowsD[s], colsD[s]);
    }
    __syncthreads();
#pragma unroll 4
    for (int e = threadIdx.x; e < nsl * bb; e += kT) {
        const int ls = e / bb, r = e - ls * bb;
        const int t = ss[ls];
        dst[base * bb + e] = (t >= 0) ? src[(int64_t)t * bb + r] : 0.0;
    }
}

__global__ void k_set_identity(int n, int b, const int *__restrict__ diag, double alpha, double *__restrict__ M)
{
    int64_t e = (int64_t)blockIdx.x * kT + threadIdx.x;
    if (e >= (int64_t)n * b) return;
    const int i = (int)(e / b), p = (int)(e - (int64_t)i * b);
    M[(int64_t)diag[i] * b * b + p * b + p] = alpha;
}

__global__ __launch_bounds__(kT) void k_fill_blocks(int64_t count, int b, const int *__restrict__ rows,
                                                    const int *__restrict__ cols, const double *__restrict__ blocks,
                                                    int natoms, const int *__restrict__ rp,
                                                    const int *__restrict__ pc, double *__restrict__ M,
                                                    int *__restrict__ bad)
{
    __shared__ int ss[kT];
    const int bb = b * b;
    const int64_t base = (int64_t)blockIdx.x * kT;
    const int nsl = (int)min((int64_t)kT, count - base);
    if (threadIdx.x < nsl) {
        const int64_t s = base + threadIdx.x;
        const int r = rows[s], c = cols[s];
        int t = -1;
        if (r >= 0 && r < natoms && c >= 0 && c < natoms) t = find_in_row(rp, pc, r, c);
        if (t < 0) atomicOr(bad, 1);
        ss[threadIdx.x] = t;
    }
    __syncthreads();
    for (int e = threadIdx.x; e < nsl * bb; e += kT) {
        const int ls = e / bb, r = e - ls * bb;
        const int t = ss[ls];
        if (t >= 0) M[(int64_t)t * bb + r] = blocks[(base + ls) * bb + r];
    }
}

}  // namespace

// whether n elements of the arrays can be read in 16-byte pairs
static bool pairs_of_16(int64_t n, const double *x, const double *y, const double *z)
{
    return n % 2 == 0 && ((reinterpret_cast<uintptr_t>(x) | reinterpret_cast<uintptr_t>(y) |
                           reinterpret_cast<uintptr_t>(z)) % 16 == 0);
}

// axpby reads pairs, except where it reads y as well and the arrays are far beyond the caches:
// single elements then stream faster.  b = 9, 10 A, beta != 0: 1000 atoms (128 MB an array) 52.1 us
// in pairs, 55.3 single; 4096 atoms (522 MB) 267 and 253; beta = 0: 35.7 and 41.0, 170 and 188.
// (Four pairs a thread with all loads first took 54, 286, 36.8 and 181.)
constexpr int64_t kSingleElements = 25000000;

void axpby(Context *ctx, int64_t n, double alpha, const double *x, double beta, double *y)
{
    if (n <= 0) return;
    if (pairs_of_16(n, x, y, y) && (beta == 0.0 || n < kSingleElements))
        k_axpby2<<<grid1(n / 2), kT, 0, ctx->stream>>>(n / 2, alpha, reinterpret_cast<const double2 *>(x), beta,
                                                       reinterpret_cast<double2 *>(y));
    else
        k_axpby<<<grid1(n), kT, 0, ctx->stream>>>(n, alpha, x, beta, y);
    BSM_HIP_TRY(hipGetLastError());
}

void axpbypcz(Context *ctx, int64_t n, double a, const double *x, double b, const double *y, double c,
              double *z)
{
    if (n <= 0) return;
    const bool paired = pairs_of_16(n, x, y, z);
    if (paired)
        k_axpbypcz2<<<grid1(n / 2), kT, 0, ctx->stream>>>(n / 2, a, reinterpret_cast<const double2 *>(x), b,
                                                          reinterpret_cast<const double2 *>(y), c,
                                                          reinterpret_cast<double2 *>(z));
    else
        k_axpbypcz<<<grid1(n), kT, 0, ctx->stream>>>(n, a, x, b, y, c, z);
    BSM_HIP_TRY(hipGetLastError());
}

void symmetrize(Context *ctx, const bsm_pattern_s *P, double *M)
{
    const int64_t n = nelems(P);
    if (n <= 0) return;
    auto go = [&](auto kern, int u) {
        kern<<<grid1((n + u - 1) / u), kT, 0, ctx->stream>>>(P->nnzb, P->b, P->tmap.as<int>(), M);
    };
    // Few elements fill the chip only one to a thread, and so do small blocks, whose threads mostly
    // end at once.  b = 9: 64 atoms, 8 A, 3.4 us with one, 4.1 with four; 216 atoms, 6 A, 4.7 and
    // 5.1; 216 atoms, 8 A, 7.7 and 7.8; 512 atoms, 16.2 and 14.3; 4096 atoms, 10 A, 248 and 227;
    // b = 3, 10 A, 34.0 and 35.7; b = 1, 16 A, 54.7 and 58.8.
    const bool one = n < (1 << 21) || P->b <= 3;
    auto block = [&](auto BC) {
        constexpr int bc = decltype(BC)::value;
        one ? go(k_symmetrize<bc, 1>, 1) : go(k_symmetrize<bc, kUnroll>, kUnroll);
    };
    if (P->b == 9) block(std::integral_constant<int, 9>{});
    else if (P->b == 4) block(std::integral_constant<int, 4>{});
    else block(std::integral_constant<int, 0>{});
    BSM_HIP_TRY(hipGetLastError());
}

void cg_update(Context *ctx, const bsm_pattern_s *P, const double *min, const double *D, const double *PN, double *L)
{
    const int64_t n = nelems(P);
    if (n <= 0) return;
    auto go = [&](auto kern) {
        kern<<<grid1((n + kUnroll - 1) / kUnroll), kT, 0, ctx->stream>>>(P->nnzb, P->b, P->tmap.as<int>(), min, D, PN,
                                                                        L);
    };
    P->b == 9 ? go(k_cg_update<9>) : P->b == 4 ? go(k_cg_update<4>) : go(k_cg_update<0>);
    BSM_HIP_TRY(hipGetLastError());
}

void add_transpose(Context *ctx, const bsm_pattern_s *P, double alpha, const double *M, double beta, double *out)
{
    const int64_t n = nelems(P);
    if (n <= 0) return;
    auto go = [&](auto kern) {
        kern<<<grid1(n), kT, 0, ctx->stream>>>(P->nnzb, P->b, P->tmap.as<int>(), alpha, M, beta, out);
    };
    P->b == 9 ? go(k_add_transpose<9>) : P->b == 4 ? go(k_add_transpose<4>) : go(k_add_transpose<0>);
    BSM_HIP_TRY(hipGetLastError());
}

void mask_copy(Context *ctx, const bsm_pattern_s *Ps, const double *src, const bsm_pattern_s *Pd, double *dst)
{
    if (Pd->nnzb <= 0) return;
    auto go = [&](auto kern, int slots) {
        kern<<<(unsigned)((Pd->nnzb + slots - 1) / slots), kT, 0, ctx->stream>>>(
            Pd->nnzb, Pd->b, Pd->rowidx.as<int>(), Pd->cols.as<int>(), Ps->rowptr.as<int>(), Ps->cols.as<int>(), src,
            dst);
    };
    auto block = [&](auto BC) {
        constexpr int bc = decltype(BC)::value;
        many_mask_slots(Pd->nnzb, Pd->b) ? go(k_mask_copy<bc, kManyMaskSlots>, kManyMaskSlots)
                                         : go(k_mask_copy<bc, kFewMaskSlots>, kFewMaskSlots);
    };
    if (Pd->b == 9) block(std::integral_constant<int, 9>{});
    else if (Pd->b == 4) block(std::integral_constant<int, 4>{});
    else block(std::integral_constant<int, 0>{});
    BSM_HIP_TRY(hipGetLastError());
}

void set_identity(Context *ctx, const bsm_pattern_s *P, double alpha, double *M)
{
    BSM_HIP_TRY(hipMemsetAsync(M, 0, sizeof(double) * (size_t)nelems(P), ctx->stream));
    const int64_t n = (int64_t)P->natoms * P->b;
    k_set_identity<<<grid1(n), kT, 0, ctx->stream>>>(P->natoms, P->b, P->diag.as<int>(), alpha, M);
    BSM_HIP_TRY(hipGetLastError());
}

void fill_blocks(Context *ctx, const bsm_pattern_s *P, double *M, int64_t count, const int32_t *rows,
                 const int32_t *cols, const double *blocks)
{
    hipStream_t st = ctx->stream;
    BSM_HIP_TRY(hipMemsetAsync(M, 0, sizeof(double) * (size_t)nelems(P), st));
    int *bad = ctx->err_flag.as<int>();
    BSM_HIP_TRY(hipMemsetAsync(bad, 0, sizeof(int), st));
    if (count > 0) {
        k_fill_blocks<<<(unsigned)((count + kT - 1) / kT), kT, 0, st>>>(
            count, P->b, rows, cols, blocks, P->natoms, P->rowptr.as<int>(), P->cols.as<int>(), M, bad);
        BSM_HIP_TRY(hipGetLastError());
    }
    int h = 0;
    BSM_HIP_TRY(hipMemcpyAsync(&h, bad, sizeof(int), hipMemcpyDeviceToHost, st));
    BSM_HIP_TRY(hipStreamSynchronize(st));
    BSM_REQUIRE(h == 0, BSM_EPATTERN, "a block falls outside the matrix pattern");
}

}  // namespace bsm
