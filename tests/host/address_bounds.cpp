// Every buffer offset that the kernels form with the address helpers of the
// library's internal header, checked against the buffers on the host.
#include <cstdio>
#include <cstring>

#include "srm3_internal.hpp"

using namespace srm3;

static int fails = 0;
#define CHECK(c, ...)                                        \
    do {                                                     \
        if (!(c)) {                                          \
            if (fails++ < 20) std::printf("FAIL " __VA_ARGS__), std::printf("\n"); \
        }                                                    \
    } while (0)

// Rows of a wave of the frequency autoconvolution: eight per tile, M in all.
static void ypair()
{
    for (int M : {1, 2, 3, 5, 7, 8, 9, 15, 16, 17, 64, 100})
        for (int q0 = 0; q0 < M; q0 += 8) {
            const int rows = M - q0 < 8 ? M - q0 : 8;
            for (int r = 0; r < 8; ++r) {
                const int x = ypair_row(r, rows);
                CHECK(x >= 0 && q0 + x < M, "ypair M %d q0 %d row %d -> %d", M, q0, r, x);
                CHECK(r >= rows || x == r, "ypair row %d of %d moved to %d", r, rows, x);
            }
        }
}

int main()
{
    ypair();
    if (!fails) std::printf("address bounds: ok\n");
    return fails != 0;
}
