// Binary32 opacity of one sample, shared by the render kernels and the
// host-side accuracy test.
#pragma once

#include <hip/hip_runtime.h>
#include <math.h>
#include <stdint.h>

namespace sqn {

// 1 - exp(-q) for q >= 0 to within 0.9 units in the last place, for small q
// too (tests/test_opacity.py; over q in [1e-9, 128] on the GPU at most 0.88
// units and 0.26 rms, as -expm1f(-q)): with
// -q = n ln 2 + r, |r| <= ln(2) / 2 and ln 2 in two parts (Cody and Waite), it
// is (1 - 2^n) - 2^n (e^r - 1), and e^r - 1 = r + r^2 p(r) with p the
// polynomial of degree 5 through (e^r - 1 - r) / r^2 at Chebyshev nodes.  n = 0,
// where 1 - 2^n vanishes, is the only case with cancellation in a direct
// evaluation.  A reduction in base 2 (r = -q log2(e) - n, whose rounding the
// series then multiplies) is off by up to 2.05 units and 0.47 rms.  Past
// q = 64 the result is 1; NaN stays NaN.
__host__ __device__ inline float opacity(float q)
{
    const float x = q > 64.0f ? -64.0f : -q;
    // adding 1.5 * 2^23 rounds to the nearest integer, which is then in the
    // low bits of the sum (a product and a sum, each with its constant in the
    // instruction: a fused one keeps one of the two in a register across the
    // march, which cost some kernels a wave)
    const float y = x * 1.44269502162933349609375f;
    const float t = y + 12582912.0f;
    const float n = t - 12582912.0f;
    float r = fmaf(n, -0.693145751953125f, x);       // 16 bits: n times it is exact
    r = fmaf(n, -1.42860682030941723212e-6f, r);
    float p = 1.98910303879529237747e-4f;
    p = fmaf(p, r, 1.39336858410388231277e-3f);
    p = fmaf(p, r, 8.33331048488616943359e-3f);
    p = fmaf(p, r, 4.16664630174636840820e-2f);
    p = fmaf(p, r, 1.66666671633720397949e-1f);
    p = fmaf(p, r, 0.5f);
    const float e = fmaf(r * r, p, r);
    uint32_t bits;
    __builtin_memcpy(&bits, &t, 4);
    bits = (bits << 23) + 0x3f800000u;               // 2^n, -93 <= n <= 0
    float s;
    __builtin_memcpy(&s, &bits, 4);
    return fmaf(-s, e, 1.0f - s);
}

}  // namespace sqn
