// Product kernels of piece scheme 1: one bf16 piece.
#include "fmt_product_kernels.h"

namespace fmt {

FMT_PRODUCT_INSTANCES(1)

}  // namespace fmt
