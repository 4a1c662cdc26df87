/* Every quotient x / s of an FP16 significand x (11 bits) by an FP32 significand s: the division that
 * the activation quantisation uses, one exact residual on top of x * y with y = 1 / s correctly
 * rounded, against the IEEE division.  Prints the number of pairs tried and of differences.
 * `step` (argument) = every how many significands of s. */
#include <stdint.h>
#include <stdio.h>
#include <stdlib.h>
#include <string.h>

int main(int argc, char **argv)
{
    const uint32_t step = argc > 1 ? (uint32_t)atoi(argv[1]) : 1;
    long long tried = 0, differ = 0;
    for (uint32_t m = 0; m < (1u << 23); m += step) {
        const uint32_t bits = 0x3f800000u | m;
        float s;
        memcpy(&s, &bits, 4);
        const float y = 1.0f / s;
        int bad = 0;
        for (int i = 1024; i < 2048; ++i) {
            const float x = (float)i, q = x * y;
            bad += __builtin_fmaf(__builtin_fmaf(-s, q, x), y, q) != x / s;
        }
        differ += bad;
        tried += 1024;
    }
    printf("%lld %lld\n", tried, differ);
    return 0;
}
