// Host-side evaluation of the scaled part of half_erfc (with 2 for its Gaussian it
// returns erfc(y) exp(y^2) for y >= 0) on arguments read from stdin; prints
// kErfNear64 first.
#include <cmath>
#include <cstdio>

#include "../paper_2108_07031_amd/csrc/qlskum_erfc.h"

int main() {
    std::printf("%.17e\n", ql::kErfNear64);
    double y;
    while (std::scanf("%lf", &y) == 1)
        std::printf("%.17e\n", ql::half_erfc(y, 2.0, 1.0 / (ql::kErfcC64 + y)));
    return 0;
}
