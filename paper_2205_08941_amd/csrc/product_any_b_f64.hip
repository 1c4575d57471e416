#define BSM_ANY_T double
#include "product_any_b.inl"

namespace bsm {
bool fits_buffers(const bsm_pattern_s *PA, const bsm_pattern_s *PB)
{
    return 8 * nelems(PA) <= (int64_t)kBufMaxBytes && 8 * nelems(PB) <= (int64_t)kBufMaxBytes;
}
}  // namespace bsm
