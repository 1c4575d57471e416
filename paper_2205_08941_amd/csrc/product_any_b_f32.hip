#define BSM_ANY_T float
#include "product_any_b.inl"
