// MFMA GEMM kernels with the QKV epilogue for rows of any sequences and positions (EPI_QKV_ROWS), tile configurations
// 0, 10, 11.
#include "gemm_mfma_impl.h"

PT_GEMM_INSTANTIATE(EPI_QKV_ROWS, 0)
PT_GEMM_INSTANTIATE(EPI_QKV_ROWS, 10)
PT_GEMM_INSTANTIATE(EPI_QKV_ROWS, 11)
