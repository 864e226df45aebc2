// MFMA GEMM kernels with the QKV epilogue for rows of any sequences and positions (EPI_QKV_ROWS), tile configurations
// 2, 9.
#include "gemm_mfma_impl.h"

PT_GEMM_INSTANTIATE(EPI_QKV_ROWS, 2)
PT_GEMM_INSTANTIATE(EPI_QKV_ROWS, 9)
