// Host-side evaluation of half_erfc_near on arguments read from stdin.
#include <cmath>
#include <cstdio>

#include "../paper_2108_07031_amd/csrc/qlskum_erfc.h"

int main() {
    std::printf("%.17e\n", ql::kErfNear64);
    double y;
    while (std::scanf("%lf", &y) == 1) std::printf("%.17e\n", ql::half_erfc_near(y));
    return 0;
}
