// Product kernels of piece scheme 0: one fp16 piece, plain and as scaled exponent planes.
#include "fmt_product_kernels.h"

namespace fmt {

FMT_PRODUCT_INSTANCES(0)
template int launch_group<0, true>(const Group &, unsigned, int, hipStream_t);

}  // namespace fmt
