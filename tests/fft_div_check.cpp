// The division by a reciprocal of the line transforms against the integer
// division, on both sides of every multiple, over the range its comment states
// (divisors up to 2^20: the rows of a field, 1024 x 1024, and less).

#include <cstdio>

#include "../paper_1012_3632_amd/csrc/fft.h"

int main() {
    long tried = 0, bad = 0;
    const int most = (1 << 22) - 2;
    for (int b = 1; b <= 1 << 20; ++b) {
        const float rb = 1.0f / (float)b;
        for (long m = 0; m <= most; m += b)
            for (long a : {m - 1, m, m + b - 1}) {
                if (a < 0 || a > most) continue;
                ++tried;
                if (flb::fft_div((int)a, rb) != (int)a / b && bad++ == 0)
                    std::printf("first: %ld / %d\n", a, b);
            }
    }
    std::printf("%ld quotients, %ld wrong\n", tried, bad);
    return bad != 0;
}
