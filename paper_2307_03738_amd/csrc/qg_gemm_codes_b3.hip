// The raw-code small-M product at 3 bits (kernels: qg_gemm_codes.h).
#define QG_CODES_KERNELS
#include "qg_gemm_codes.h"

int qg_codes_launch_b3(int gps, int mb, const QgCodesArgs &A, int workgroups, hipStream_t st, QgKernelInfo *query)
{
    return codes_launch_any<3>(gps, mb, A, workgroups, st, query);
}

void qg_codes_prepare_b3(const QgPrepArgs &P, int rows_padded, hipStream_t st) { codes_prepare<3>(P, rows_padded, st); }
