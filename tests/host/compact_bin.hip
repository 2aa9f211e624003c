// compact_bin stays within the quantile table, with no conversion out of range
// (host code only; no device work)
#include <cmath>
#include <cstdio>
#include <limits>

#include "k_search.hpp"

int main()
{
    const float inf = std::numeric_limits<float>::infinity(), tiny = std::numeric_limits<float>::denorm_min();
    const float big = std::numeric_limits<float>::max();
    const float outside[] = {NAN, -NAN, inf, -inf, big, -big, 1e10f, -1e10f, 3e9f / 256, -3e9f / 256, 1.f, 2.f, -1.f, 0.f, -0.f};
    int bad = 0;
    for (float A : outside) {
        const int b = peos::compact_bin(A);
        const int want = A >= 1.f ? peos::kCompactLutBins - 1 : 0;
        if (b != want) bad += std::printf("A=%g: bin %d\n", (double)A, b) > 0;
    }
    for (float A = tiny; A < 1.f; A = A < 1e-6f ? A * 3.f : A + 1.f / 4099) {
        const int b = peos::compact_bin(A);
        if (b != (int)((double)A * peos::kCompactLutBins)) bad += std::printf("A=%g: bin %d\n", (double)A, b) > 0;
    }
    if (peos::compact_bin(std::nextafter(1.f, 0.f)) != peos::kCompactLutBins - 1) ++bad;
    std::printf(bad ? "compact bin failed\n" : "compact bin ok\n");
    return bad != 0;
}
