// The bf16 kernels of kernels_conv_rows.hip.
#define WMDEC_CONV_ROWS_BF16
#include "kernels_conv_rows.hip"
