// The padding rule of set_geometry (linked with the built library, no GPU):
// every length it returns holds the convolution, and a 3D axis grows only as
// far as the column passes without compiled kernels can bear (built by
// tests/test_host_runtime.py).
#include <stdio.h>

#include "host_common.hpp"

using namespace llg;
using namespace llg::host;

static int failures = 0;

static void lengths(const int n[3], const int pb[3], int P0[3], int P[3]) {
    for (int a = 0; a < 3; ++a) P[a] = P0[a] = n[2] == 1 && a == 2 ? 1 : pb[a] ? n[a] : pad_len(n[a]);
    compiled_lengths(n, pb, P);
}

static void expect(int nx, int ny, int nz, int px, int py, int pz) {
    const int n[3] = {nx, ny, nz}, pb[3] = {0, 0, 0};
    int P0[3], P[3];
    lengths(n, pb, P0, P);
    if (P[0] != px || P[1] != py || P[2] != pz) {
        ++failures;
        fprintf(stderr, "%d x %d x %d cells: %d x %d x %d points, not %d x %d x %d\n", nx, ny, nz, P[0], P[1], P[2], px, py,
                pz);
    }
}

int main() {
    // z at runtime length (above 256 planes): y and x almost as short as they can be
    expect(4, 600, 300, 8, 1200, 600);
    expect(34, 40, 300, 70, 96, 600);
    expect(300, 20, 270, 600, 40, 540);
    expect(64, 17, 300, 128, 36, 600);
    expect(125, 40, 300, 256, 96, 600);
    expect(650, 40, 300, 1536, 96, 600);
    expect(540, 40, 300, 1080, 96, 600);
    // y alone at runtime length (above 512 cells)
    expect(10, 1000, 20, 20, 2000, 48);
    expect(100, 600, 20, 200, 1200, 48);
    expect(540, 600, 20, 1536, 1200, 48);
    expect(24, 600, 4, 64, 1200, 8);
    // as many points as a launch may have threads: as it is
    expect(980, 1000, 540, 1960, 2000, 1080);
    // every pass compiled
    expect(4, 100, 20, 64, 256, 48);
    expect(100, 60, 20, 256, 128, 48);
    expect(600, 512, 256, 1536, 1024, 512);
    expect(1000, 600, 1, 2048, 1536, 1);
    expect(1000, 1030, 1, 2048, 4096, 1);
    const int sx[] = {1, 2, 3, 5, 18, 33, 60, 100, 257, 500, 520, 700, 1000, 1024};
    const int sy[] = {1, 2, 4, 18, 40, 75, 100, 250, 500, 512, 600, 1000, 2048};
    const int sz[] = {1, 2, 3, 8, 9, 20, 60, 135, 250, 256, 270, 300, 1000};
    long long cases = 0;
    for (int nx : sx)
        for (int ny : sy)
            for (int nz : sz)
                for (int m = 0; m < 8; ++m) {
                    const int n[3] = {nx, ny, nz}, pb[3] = {m & 1, m >> 1 & 1, m >> 2 & 1};
                    bool ok = true;
                    for (int a = 0; a < 3; ++a) ok = ok && (!pb[a] || good_len(n[a]));
                    if (!ok || (pb[0] && nx % 2) || (nz == 1 && pb[2])) continue;
                    int P0[3], P[3];
                    lengths(n, pb, P0, P);
                    ++cases;
                    for (int a = 0; a < 3; ++a) ok = ok && P[a] >= P0[a] && (P[a] == P0[a] || P[a] >= 2 * n[a] - 1);
                    if (nz > 1) {
                        const int split = !pb[2] || P[2] != P0[2];
                        const bool zfast = fast3d_col_ok(P[2], split, true) || fast3d_thin_ok(nz, P[2], split);
                        const bool yfast = fast3d_col_ok(P[1], !pb[1] || P[1] != P0[1], false);
                        if (!zfast) ok = ok && P[1] <= 1.25 * P0[1] && P[0] <= 1.2 * P0[0];
                        if (!yfast && P0[0] <= 1024 && (P[0] / 2 + 1) * nz > 200) ok = ok && P[0] <= 1.05 * P0[0];
                    }
                    if (!ok) {
                        ++failures;
                        fprintf(stderr, "%d x %d x %d cells, periodic %d: %d x %d x %d points\n", nx, ny, nz, m, P[0], P[1],
                                P[2]);
                    }
                }
    if (failures) return 1;
    printf("padding ok (%lld)\n", cases);
    return 0;
}
