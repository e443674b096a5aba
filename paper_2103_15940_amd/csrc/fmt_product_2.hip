// Product kernels of piece scheme 2: two bf16 pieces.
#include "fmt_product_kernels.h"

namespace fmt {

FMT_PRODUCT_INSTANCES(2)

}  // namespace fmt
