// Row passes with a key product, primes below 2^60 (signed Montgomery products).
#include "kernels_impl.hpp"

namespace nttk {
// row passes: instantiated in kernels_rows.hip
#define X(LM) NTTK_MUL_ROWS(extern, true, LM, false) NTTK_MUL_ROWS(extern, true, LM, true)
NTTK_ROW_CASES(X)
#undef X
template hipError_t mul_rows<true>(const PassArgs&, const PassArgs&, int, hipStream_t);
}  // namespace nttk
