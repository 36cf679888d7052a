/* Checks of two fp32 identities the int8 epilogues rely on (IEEE binary32, round to nearest even,
 * denormals kept):
 *   div127:  x * RN(1/127) corrected once by fma from its exact remainder equals the
 *            correctly rounded x / 127, for every non-negative finite x;
 *   code:    the low byte of fma(x, r, M), M = 1.5 * 2^23, clamped to [M + lo, M + 127], is the
 *            two's complement of the exact product x r rounded half to even and clamped to
 *            [lo, 127].  lo = -127 for every x of either sign up to a block's largest, lo = 1 and
 *            0 for the non-negative ones; r is the reciprocal of the block's scale, or one of its
 *            two neighbours (the hardware's reciprocal is good to 1 ulp), so that products land
 *            on both sides of 127 and, for scales that are powers of two, on exact ties.  The
 *            product of two floats is exact in a double.
 * Prints the number of mismatches of each; exit status 0 when both are zero. */
#include <math.h>
#include <stdint.h>
#include <stdio.h>
#include <string.h>

static float as_float(uint32_t b) { float f; memcpy(&f, &b, 4); return f; }
static uint32_t as_bits(float f) { uint32_t b; memcpy(&b, &f, 4); return b; }

/* v_med3_f32 of three finite values, the second and third in order */
static float median(float x, float lo, float hi) { return x < lo ? lo : x > hi ? hi : x; }

static int code_differs(float x, float r, float lo)
{
    const float M = 12582912.0f;
    const uint8_t got = (uint8_t)(as_bits(median(fmaf(x, r, M), M + lo, M + 127.0f)) & 0xFFu);
    double y = rint((double)x * (double)r);
    y = y < lo ? lo : y > 127.0 ? 127.0 : y;
    return got != (uint8_t)(int8_t)(int)y;
}

int main(void)
{
    const float R = 1.0f / 127.0f;
    long long bad_div = 0, bad_code = 0;
#pragma omp parallel for reduction(+ : bad_div) schedule(static)
    for (long long u = 0; u < 0x7F800000LL; ++u) {
        const float x = as_float((uint32_t)u);
        const volatile float q = x * R;
        const float s = fmaf(fmaf(-q, 127.0f, x), R, q);
        const volatile float t = x / 127.0f;
        if (as_bits(s) != as_bits(t)) ++bad_div;
    }
    const float amax[] = {127.0f, 3.3e-4f, 1.7e-6f, 0x1.fffffep+3f, 9.9e-30f};
    for (unsigned k = 0; k < sizeof amax / sizeof amax[0]; ++k) {
        const float s = amax[k] / 127.0f, r0 = 1.0f / s;
        const uint32_t top = as_bits(amax[k]);
        for (int ulp = -1; ulp <= 1; ++ulp) {
            const float r = as_float(as_bits(r0) + (uint32_t)ulp);
            /* codes 0 to 127 lie in the top ten binades: every value there, every 97th below */
            const long long low = (long long)top - (10LL << 23), from = low > 0 ? low : 0;
#pragma omp parallel for reduction(+ : bad_code) schedule(static)
            for (long long u = from; u <= (long long)top; ++u) {
                const float x = as_float((uint32_t)u);
                bad_code += code_differs(x, r, -127.0f) + code_differs(-x, r, -127.0f) + code_differs(x, r, 1.0f);
            }
#pragma omp parallel for reduction(+ : bad_code) schedule(static)
            for (long long u = 0; u < from; u += 97) {
                const float x = as_float((uint32_t)u);
                bad_code += code_differs(x, r, -127.0f) + code_differs(-x, r, -127.0f) + code_differs(x, r, 1.0f);
            }
        }
    }
    bad_code += code_differs(0.0f, 0.0f, 0.0f) + code_differs(0.0f, 0.0f, -127.0f);   /* a block of zeros */
    printf("div127 %lld code %lld\n", bad_div, bad_code);
    return bad_div || bad_code;
}
