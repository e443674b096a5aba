// Product kernels of the convolutions on exponent planes: one fp16 piece, one scale per operand.
#include "fmt_product_kernels.h"

namespace fmt {

template int product_window<false>(const OperandView &, const OperandView &, const Implicit &, int, int, int, const OutSpec &, const Plan &, float *,
                                   hipStream_t);
template int product_window<true>(const OperandView &, const OperandView &, const Implicit &, int, int, int, const OutSpec &, const Plan &, float *,
                                  hipStream_t);

}  // namespace fmt
