// Internal to libktanh: the approximants of TanH that K-TanH is compared with, on one Float32 magnitude.
// Plain C++ (no device headers) so that host tests can evaluate them over all inputs.
#pragma once

#ifdef __HIPCC__
#define KT_APPROX __host__ __device__ inline
#else
#define KT_APPROX inline
#endif

namespace ktanh_device {

// Pade[3/2] = x (15 + x^2) / (15 + 6 x^2) on min(|x|, 4), capped at 1;
// Pade[7/8] = x (2027025 + 270270 x^2 + 6930 x^4 + 36 x^6) / (2027025 + 945945 x^2 + 51975 x^4 + 630 x^6 + x^8)
// on min(|x|, 5.5).  `a` is the clamped magnitude, `rcp` the reciprocal.
// Float32, Horner's scheme in x^2 with fused multiply-adds, and the numerator times the hardware's reciprocal
// of the denominator.  With one rounding per operation and a correctly rounded division (the definition, and
// what this was before) the kernels ran at the rate of the vector units: a division alone is ten
// instructions.  The BFloat16 result is the same for every one of the 2^16 inputs, and it stays the same with
// the reciprocal moved by up to two units in its last place (the hardware's is within one).  us per launch
// before -> now: Pade[7/8] 24.6 -> 16.3 on [6400, 4096], 120.9 -> 79.9 on [8192, 16384]; Pade[3/2] 19.8 -> 16.0,
// 94.4 -> 77.1; K-TanH, which is the memory stream, 15.9 and 77.1.
template <bool SEVEN_EIGHT, class Reciprocal>
KT_APPROX float pade_of_magnitude(float a, Reciprocal rcp)
{
    const float x2 = a * a;
    if constexpr (SEVEN_EIGHT) {
        float p = __builtin_fmaf(36.0f, x2, 6930.0f);
        p = __builtin_fmaf(p, x2, 270270.0f);
        p = __builtin_fmaf(p, x2, 2027025.0f);
        float q = x2 + 630.0f;
        q = __builtin_fmaf(q, x2, 51975.0f);
        q = __builtin_fmaf(q, x2, 945945.0f);
        q = __builtin_fmaf(q, x2, 2027025.0f);
        return (a * p) * rcp(q);
    } else {
        const float y = (a * (15.0f + x2)) * rcp(__builtin_fmaf(6.0f, x2, 15.0f));
        return __builtin_fminf(y, 1.0f);
    }
}

// The Taylor polynomial of TanH about the midpoint a of K-TanH's interval, at a + h, from y = TanH(a) alone:
// the derivatives over k! are  d = 1 - y^2,  -y d,  -d (1 - 3 y^2) / 3,  so
//   degree 2:  y + (h d) (1 - h y)          degree 3:  y + (h d) (1 - h (y + h (1/3 - y^2))).
// One cross-lane table read per element, as K-TanH itself has; with the three or four coefficients read from
// a table (rounded to Float32 on the host) the cross-lane unit was busy for longer than the stream takes.
// The BFloat16 result is the same for every one of the 2^16 inputs.  us per launch before -> now: degree 2
// 19.5 -> 16.3 on [6400, 4096], 90.6 -> 77.7 on [8192, 16384]; degree 3 22.6 -> 16.4, 108.9 -> 79.8.
template <int DEGREE>
KT_APPROX float taylor_at(float h, float y)
{
    const float hd = h * __builtin_fmaf(-y, y, 1.0f);
    float inner = y;
    if constexpr (DEGREE == 3) inner = __builtin_fmaf(h, __builtin_fmaf(-y, y, 1.0f / 3.0f), y);
    return __builtin_fmaf(hd, __builtin_fmaf(-h, inner, 1.0f), y);
}

}  // namespace ktanh_device
