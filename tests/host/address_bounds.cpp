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

// Operand of the split-FP16 pair sum: the 16 bytes that a block stages of any
// start lie in it, in every column; those it may use are the rows they stand
// for; and the operand fits the region the workspace keeps for it (three FP32
// values per support column and row, rows padded to the rows per wave).
static void split()
{
    for (int nk = 32; nk <= 700; ++nk) {
        const int rs = nk <= 64 ? 64 : (nk <= 128 ? 128 : 256);
        const unsigned col_bytes = static_cast<unsigned>(split_seg(nk)) * 8u;
        for (int ncw : {1, 3, 2047})
            for (int R : {2, 4, 8, 16}) {
                const size_t nkp = static_cast<size_t>((nk + R - 1) / R * R);
                CHECK(split_operand_bytes(nk, ncw) <= 12 * ncw * nkp, "split nk %d ncw %d R %d: operand", nk, ncw, R);
            }
        for (int p = 0; p < 8; ++p)
            for (int k = -2 * rs - 8; k <= nk + 2 * rs; ++k) {
                const unsigned o = split_start(nk, p, k);
                for (int ncw : {1, 9})
                    CHECK((ncw - 1) * static_cast<size_t>(col_bytes) + o + 16 <= split_operand_bytes(nk, ncw),
                          "split nk %d part %d row %d: offset %u in the last of %d columns", nk, p, k, o, ncw);
                if (p < 4 && k > -8 && k < nk)
                    CHECK(o == static_cast<unsigned>(p * split_seg(nk) + 8 + k) * 2u, "split nk %d part %d row %d", nk, p, k);
                else if (p < 4 && k >= split_nk8(nk))
                    CHECK(o == 0, "split nk %d part %d row %d is past the rows", nk, p, k);
            }
    }
}

// Work items of the FP64 matrix-core pair sum are counted in 32 bits: at the
// largest grids and batches the library takes (2^31 lines a call, 65535
// realizations), with tiles of 32 x 32 outputs and less, in chunks of at least
// 16 partners.
static void queue()
{
    for (long nk : {1L, 2L, 3L, 16L, 100L, 4096L})
        for (long nc : {1L, 63L, 8191L})
            for (long rows : {32L, 16L})
                for (long cols : {32L, 16L}) {
                    const long tiles = ((nk + rows - 1) / rows) * ((nc + cols - 1) / cols);
                    const long chunks = nc / 16 + 1;
                    const long batch = (1L << 31) / (nk * nc) < 65535 ? (1L << 31) / (nk * nc) : 65535;
                    const long per = mfma_queue_batch(tiles * chunks);
                    CHECK(per >= 1 && (per < batch ? per : batch) * tiles * chunks < (1L << 31) - 4096,
                          "queue %ldx%ld: %ld realizations of %ld items in a launch", nk, nc, per, tiles * chunks);
                }
}

int main()
{
    queue();
    ypair();
    split();
    if (!fails) std::printf("address bounds: ok\n");
    return fails != 0;
}
