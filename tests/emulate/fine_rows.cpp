// The rows that Ep holds for partial outputs per 64 units are the most list entries whose launch
// writes such outputs, for every width, token count and grid.
#include "k_epsnet.hip"

using namespace pa;

template <int H>
static int check(int ntok, int grid) {
    int most = 0;                       // list entries: no launch of more than grid 32-token slices
    for (int m = 1; m <= grid; ++m) {
        const int c = fine_choice<H>(m, ntok, 1 << 30, grid);
        if (c == FINE_32x128 || c == FINE_32x256) most = m;
    }
    const int rows = mlp_fine_rows(H, ntok, grid);
    if (rows == most) return 0;
    printf("FAILED: H %d, %d tokens, %d blocks: %d rows for at most %d list entries\n", H, ntok, grid, rows, most);
    return 1;
}

int main() {
    int bad = 0;
    for (int grid : {256, 304, 120, 64, 8})
        for (int ntok = 128; ntok <= 65536; ntok += ntok < 4096 ? 128 : 4096)
            bad += check<512>(ntok, grid) + check<1024>(ntok, grid) + check<2048>(ntok, grid);
    if (!bad) printf("fine rows ok\n");
    return bad != 0;
}
