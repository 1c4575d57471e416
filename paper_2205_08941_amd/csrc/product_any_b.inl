// The kernel and launcher of product_any_b.h for operands of type BSM_ANY_T.
//
// The tile of product.hip's ring kernels with the block size as a parameter: b = 13 (two
// radial functions each for s and p, one for d) in blocks of 1352 bytes, 4 rows x 4
// columns.  It replaces the scalar-operand kernel, which waits for every A block to come
// through the scalar cache: 480 atoms, b = 13, 10 A x 6 A -> 16 A took 4.84 ms there and
// takes 0.92 here.
#include "product_any_b.h"
#include "tiles.h"

namespace bsm {
namespace {

constexpr int kXcds = 8;

template <int B, int G, class T, int TR>
__global__ __launch_bounds__(64) void k_product_ring_any(
    int64_t ntiles, int64_t nwg_padded, const int *__restrict__ order, const int *__restrict__ hdr,
    const int64_t *__restrict__ ebeg, const int *__restrict__ ent, const T *__restrict__ vA, const T *__restrict__ vB,
    const T *__restrict__ zblk, double *__restrict__ vC, double alpha, double beta, unsigned a_bytes, unsigned b_bytes)
{
    __shared__ __attribute__((aligned(16))) char ring[2 * RingEntry<B, G, T>::kStep];
    const int64_t w = blockIdx.x, t = (w % kXcds) * (nwg_padded / kXcds) + w / kXcds;
    if (t >= ntiles) return;
    tile_ring<B, G, 2, T, kBufferCopies, 1, TR>(order[t], hdr, ebeg, ent, vA, vB, zblk, vC, alpha, beta,
                                                (lds_char_t *)ring, a_bytes, b_bytes);
}

template <int B, int G>
void launch_rows(hipStream_t st, const Plan *plan, const BSM_ANY_T *A, const BSM_ANY_T *Bm, double *C, double alpha,
                double beta, const BSM_ANY_T *zblk, int64_t a_bytes, int64_t b_bytes)
{
    const int64_t nwg_padded = ((plan->ntiles + kXcds - 1) / kXcds) * kXcds;
    auto go = [&](auto kern, const BSM_ANY_T *x, int64_t xb, const BSM_ANY_T *y, int64_t yb) {
        kern<<<(unsigned)nwg_padded, 64, 0, st>>>(plan->ntiles, nwg_padded, plan->order.as<int>(),
                                                  plan->hdr.as<int>(), plan->ebeg.as<int64_t>(), plan->ent.as<int>(),
                                                  x, y, zblk, C, alpha, beta, (unsigned)xb, (unsigned)yb);
    };
    // a transposed plan's row operand is B
    if (plan->transposed) go(k_product_ring_any<B, G, BSM_ANY_T, 1>, Bm, b_bytes, A, a_bytes);
    else go(k_product_ring_any<B, G, BSM_ANY_T, 0>, A, a_bytes, Bm, b_bytes);
}

template <int B>
void launch_any(hipStream_t st, const Plan *plan, const BSM_ANY_T *A, const BSM_ANY_T *Bm, double *C, double alpha,
                double beta, const BSM_ANY_T *zblk, int64_t a_bytes, int64_t b_bytes)
{
    if (plan->G == 2) launch_rows<B, 2>(st, plan, A, Bm, C, alpha, beta, zblk, a_bytes, b_bytes);
    else launch_rows<B, (B <= 8 ? 8 : 4)>(st, plan, A, Bm, C, alpha, beta, zblk, a_bytes, b_bytes);
}

}  // namespace

void launch_any_b(hipStream_t st, const Plan *plan, const BSM_ANY_T *A, const BSM_ANY_T *B, double *C, double alpha,
                  double beta, const BSM_ANY_T *zblk, int64_t a_bytes, int64_t b_bytes)
{
    BSM_REQUIRE(plan->variant == 4 && plan->waves == 1 && (plan->G == 2 || plan->G == any_b_rows(plan->b, false)) &&
                    a_bytes <= (int64_t)kBufMaxBytes && b_bytes <= (int64_t)kBufMaxBytes,
                BSM_EINVAL, "not a ring plan of this block size");
    switch (plan->b) {
#define X(b) \
    case b: launch_any<b>(st, plan, A, B, C, alpha, beta, zblk, a_bytes, b_bytes); break;
        X(5) X(6) X(7) X(8) X(10) X(11) X(12) X(13) X(14) X(15) X(16)
#undef X
        default: throw Error{BSM_EINVAL, "no ring kernel for this b"};
    }
}

}  // namespace bsm
