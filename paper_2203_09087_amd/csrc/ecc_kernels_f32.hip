// The histogram kernels for float32 data (ecc_kernels_dt.h).
#define ECC_KERNEL_DT DT_F32
#include "ecc_kernels_dt.h"
