// The rows that the blocks of the inverse row kernel stage, for every number
// of row pairs per block and film height, without a GPU (built by
// tests/test_host_runtime.py): each row read lies inside the film, and each
// owned row and its y neighbours are staged as they are (or as zeros where an
// open film ends).
#include <stdio.h>
#include <stdlib.h>

#include "internal.hpp"

using namespace llg;

int main() {
    long long bad = 0, n = 0;
    for (int RP = 1; RP <= 32; RP *= 2) {      // 64 lanes / lanes per transform (2 ... 64)
        const int NR = 2 * RP + 2;
        for (int ny = 1; ny <= 4 * RP + 3; ++ny)
            for (int wrap = 0; wrap < 2; ++wrap)
                for (int rb = 0; rb < ny; rb += 2 * RP) {
                    for (int rq = 0; rq < NR; ++rq, ++n) {
                        bool ok = false;
                        const int row = staged_row(rb - 1 + rq, ny, wrap != 0, ok);
                        if (ok && (row < 0 || row >= ny)) {
                            if (bad++ < 10)
                                fprintf(stderr, "RP %d ny %d wrap %d block %d: staged row %d is row %d\n", RP, ny, wrap, rb,
                                        rq, row);
                        }
                    }
                    for (int r = rb; r < ny && r < rb + 2 * RP; ++r)
                        for (int d = -1; d <= 1; ++d) {
                            bool ok = false;
                            const int row = staged_row(r + d, ny, wrap != 0, ok);
                            const bool in = r + d >= 0 && r + d < ny;
                            if (ok != (in || wrap) || (ok && row != (r + d + ny) % ny)) {
                                if (bad++ < 10) fprintf(stderr, "RP %d ny %d wrap %d row %d%+d: %d\n", RP, ny, wrap, r, d, row);
                            }
                        }
                }
    }
    if (bad) return 1;
    printf("staged rows ok (%lld)\n", n);
    return 0;
}
