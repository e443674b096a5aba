// Product kernels of piece scheme 3: three bf16 pieces.
#include "fmt_product_kernels.h"

namespace fmt {

FMT_PRODUCT_INSTANCES(3)

}  // namespace fmt
