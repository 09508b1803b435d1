// The layout kernel of the Python operations' host side (shv_host.cpp).
#pragma once

#include <stdint.h>

#include "shvis.h"

#ifdef __cplusplus
extern "C" {
#endif

// a, b [P][3] -> oa, ob [3][P], in one launch.
shv_status shv_internal_soa(const float* a, const float* b, int64_t P, float* oa, float* ob, hipStream_t stream);

#ifdef __cplusplus
}
#endif
