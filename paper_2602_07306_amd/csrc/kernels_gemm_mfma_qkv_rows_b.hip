// MFMA GEMM kernels with the QKV epilogue for rows of any sequences and positions (EPI_QKV_ROWS), tile configurations
// 1, 4, 8.
#include "gemm_mfma_impl.h"

PT_GEMM_INSTANTIATE(EPI_QKV_ROWS, 1)
PT_GEMM_INSTANTIATE(EPI_QKV_ROWS, 4)
PT_GEMM_INSTANTIATE(EPI_QKV_ROWS, 8)
