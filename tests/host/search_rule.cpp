// The rule that gives a clip search to its grid form, asked for each line of the input: rows n bits sylvester waves
// rows_per_pass threads steps, the device's LDS in bytes and what of it is taken.  Prints 1 (grid) or 0 a line.
#include <cstdio>

#include "../../paper_2504_13989_amd/csrc/search_rule.h"

int main() {
    long long rows, lds, taken;
    int n, bits, sylvester, waves, rpp, threads, steps;
    while (std::scanf("%lld %d %d %d %d %d %d %d %lld %lld", &rows, &n, &bits, &sylvester, &waves, &rpp, &threads, &steps,
                      &lds, &taken) == 10) {
        const rq::GridCase c{rows, n, bits, 256, sylvester != 0, rq::grid_rows_beside(bits, lds, taken), waves, rpp, threads};
        std::printf("%d\n", rq::gbs_grid_pays(c, steps) ? 1 : 0);
    }
    return 0;
}
