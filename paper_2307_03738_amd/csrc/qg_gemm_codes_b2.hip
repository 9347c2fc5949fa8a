// The raw-code small-M product at 2 bits (kernels: qg_gemm_codes.h).
#define QG_CODES_KERNELS
#include "qg_gemm_codes.h"

int qg_codes_launch_b2(int gps, int mb, const QgCodesArgs &A, int workgroups, hipStream_t st, QgKernelInfo *query)
{
    return codes_launch_any<2>(gps, mb, A, workgroups, st, query);
}

void qg_codes_prepare_b2(const QgPrepArgs &P, int rows_padded, hipStream_t st) { codes_prepare<2>(P, rows_padded, st); }
