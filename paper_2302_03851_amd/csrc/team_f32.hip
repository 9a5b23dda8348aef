// Team kernels of the fp32 chain, lattice and child-sum cells.
#include <hip/hip_runtime.h>

#include <type_traits>

#include "team.h"
#include "team_table.h"

using namespace edbk;

edb::TeamEntry edb::team_entry_f32(int family, int nk) {
    switch (family) {
        case TF_CHAIN: return pick<float, 1, K_CHAIN, -1, 1, 2, 3, 4, 5, 8>(nk);
        case TF_LATTICE: return pick<float, 1, K_LAT_CHAR, K_LAT_WORD, 1, 2, 3, 4>(nk);
        case TF_LGRU: return pick<float, 1, K_LGRU_EDGE, K_POOL_MEAN, 1, 2, 3, 4, 5>(nk);
        case TF_CHILDSUM: return pick<float, 1, K_CS_INT, -1, 1, 2, 3, 4>(nk);
        default: return {};
    }
}
