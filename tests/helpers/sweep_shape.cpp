// Prints the sweep shape that the library gives an instance, host only:
//   sweep_shape DIM REAL L R SWEEPS TILE_ROWS GROUP_REPLICAS ...  (seven numbers a line of output)
// as "status replicas_per_word sets tile_rows group_replicas blocks_of_a_colour".
#include <cstdio>
#include <cstdlib>
#include <vector>

#include "../../paper_1710_09025_amd/csrc/runner.h"

namespace pamc {
int make_inst(int L, const int8_t *J, const int32_t *Jq, int64_t R, const double *beta, int nT, int NS,
              uint64_t seed, const pamc_options &opt, HostInst &h);
}

int main(int argc, char **argv)
{
    for (int i = 1; i + 7 <= argc; i += 7) {
        const int dim = atoi(argv[i]), real = atoi(argv[i + 1]), L = atoi(argv[i + 2]);
        pamc_options o;
        pamc_default_options(&o);
        o.dim = dim;
        o.tile_rows = atoi(argv[i + 5]);
        o.group_replicas = atoi(argv[i + 6]);
        size_t n = dim;
        for (int d = 0; d < dim; ++d) n *= L;
        const std::vector<int8_t> J(n, 1);
        const std::vector<int32_t> Jq(n, 1);
        const double beta[2] = {0.0, 1.0};
        pamc::HostInst h;
        const int st = pamc::make_inst(L, J.data(), real ? Jq.data() : nullptr, atoll(argv[i + 3]), beta, 2,
                                       atoi(argv[i + 4]), 1, o, h);
        printf("%d %d %d %d %d %d\n", st, h.mrep, h.sets, h.tile_rows, 4 * h.rp, h.gmax);
    }
    return 0;
}
