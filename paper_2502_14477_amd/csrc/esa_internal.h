// Exported beside the boundary of esa.h, for the tests: nothing else calls it, and it may change with the kernels.
#pragma once
#include "esa.h"

extern "C" {

// esa_score whose workgroups wait at most ticks * 10 ns for one another before they do the missing work themselves.
ESA_API int esa_internal_score_waiting(const void* qc, int l_c, const void* kc_cache, int64_t m_lo, int64_t m_hi, int d_c, int eps,
                                       float* score, int dtype, int batch, int64_t q_bs, int64_t kc_bs, int64_t score_bs, void* workspace,
                                       size_t ws_bytes, uint32_t ticks, void* stream);

}  // extern "C"
