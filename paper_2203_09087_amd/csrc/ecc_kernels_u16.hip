// The histogram kernels for uint16 data (ecc_kernels_dt.h).
#define ECC_KERNEL_DT DT_U16
#include "ecc_kernels_dt.h"
