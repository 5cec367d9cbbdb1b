// The histogram kernels for uint8 data (ecc_kernels_dt.h).
#define ECC_KERNEL_DT DT_U8
#include "ecc_kernels_dt.h"
