// Shared by the fp32 kernels: log2(e) and a row's LSE in units of log2, as two floats each.
#pragma once
#include "hexi_internal.h"
#include "hexi_mfma.h"

namespace {

constexpr float LOG2E_HI = 1.44269502162933349609f;      // log2(e) rounded to fp32, and the rest
constexpr float LOG2E_LO = 1.92596299112661746887e-8f;

// -LSE * log2(e) as two floats.  A row whose LSE is infinite (one that sees nothing anywhere, or that is switched off) has P = 0.
__device__ __forceinline__ void neg_lse_log2(float l, float& hi, float& lo)
{
    const bool live = fabsf(l) != INFINITY;
    hi = live ? -l * LOG2E_HI : -INFINITY;
    lo = live ? fmaf(-l, LOG2E_HI, -hi) - l * LOG2E_LO : 0.f;
}

}  // namespace
