/* The shortcut of the row quantisers (RowQuantizer::packed8_own_max), written out for the host: for fp16 row maxima and every fp16
 * value up to them, a value that the shortcut keeps must have the code of the definition, rne(fl32(x / scale)).  Prints the number of
 * pairs, of pairs whose quotient is a half-integer, and of wrong codes and of values sent to the division for the margin of the row
 * maximum and the margin per value.  TIE_MARGIN, TIE_REST: the kernels' constants kTieMargin and kTieRest, given to the compiler.
 * usage: quotient_margin qmax first step   (row maxima first, first + step, ... of the positive finite fp16 values, by bit pattern) */
#include <math.h>
#include <stdint.h>
#include <stdio.h>
#include <stdlib.h>

static float half_value(unsigned h) {
    const int e = (int)(h >> 10), m = (int)(h & 1023u);
    return e == 0 ? ldexpf((float)m, -24) : ldexpf((float)(m + 1024), e - 25);
}

int main(int argc, char **argv) {
    if (argc != 4) return 2;
    const float qmax = (float)atoi(argv[1]), shift = 12582912.0f, c = TIE_MARGIN;
    const unsigned first = (unsigned)atoi(argv[2]), step = (unsigned)atoi(argv[3]);
    static float value[0x7C00];
    for (unsigned h = 0; h < 0x7C00u; ++h) value[h] = half_value(h);
    unsigned long long pairs = 0, halves = 0, wrong[2] = {0, 0}, sent[2] = {0, 0};
#pragma omp parallel for schedule(dynamic, 8) reduction(+ : pairs, halves, wrong[:2], sent[:2])
    for (unsigned a = first; a < 0x7C00u; a += step) {
        const float scale = value[a] / qmax, recip = 1.0f / scale, margin = qmax * c;
        for (unsigned h = 0; h <= a; ++h) {
            const float x = value[h], t = fmaf(x, recip, shift), n = t - shift, distance = fabsf(fmaf(x, recip, shift - t));
            const int keep[2] = {!(distance > 0.5f - margin), !(fmaf(fabsf(shift - t), c, distance) > 0.5f - TIE_REST)};
            const int differs = n != rintf(x / scale);
            const double twice = 2.0 * (double)x * (double)qmax / (double)value[a];  /* exact where it is an integer */
            halves += twice == rint(twice) && fmod(twice, 2.0) == 1.0;
            for (int i = 0; i < 2; ++i) {
                sent[i] += !keep[i];
                wrong[i] += keep[i] && differs;
            }
            ++pairs;
        }
    }
    printf("%llu %llu %llu %llu %llu %llu\n", pairs, halves, wrong[0], wrong[1], sent[0], sent[1]);
    return 0;
}
