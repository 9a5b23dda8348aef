// Team kernels of the bf16 cells (one or two unit blocks a work-group).
#include <hip/hip_runtime.h>

#include <type_traits>

#include "team.h"
#include "team_table.h"

using namespace edbk;

edb::TeamEntry edb::team_entry_bf16(int family, int nk, int ub) {
    if (ub == 1) {
        switch (family) {
            case TF_CHAIN: return pick<__bf16, 1, K_CHAIN, -1, 1, 2, 3>(nk);
            case TF_NARY: return pick<__bf16, 1, K_NARY_INT, -1, 1, 2, 3>(nk);
            case TF_NARY2: return pick<__bf16, 1, K_NARY_INT, K_NARY_INT, 1, 2, 3>(nk);
            case TF_GRU: return pick<__bf16, 1, K_GRU_INT, -1, 1, 2, 3>(nk);
            case TF_GRID: return pick<__bf16, 1, K_GRID, -1, 1, 2, 3, 4>(nk);
            case TF_LATTICE: return pick<__bf16, 1, K_LAT_CHAR, K_LAT_WORD, 1, 2, 3>(nk);
            case TF_CHILDSUM: return pick<__bf16, 1, K_CS_INT, -1, 1>(nk);
            default: return {};
        }
    }
    switch (family) {
        case TF_CHAIN: return pick<__bf16, 2, K_CHAIN, -1, 2, 3, 4>(nk);
        case TF_NARY: return pick<__bf16, 2, K_NARY_INT, -1, 3, 4>(nk);
        case TF_GRU: return pick<__bf16, 2, K_GRU_INT, -1, 3, 4>(nk);
        case TF_LATTICE: return pick<__bf16, 2, K_LAT_CHAR, K_LAT_WORD, 2>(nk);
        case TF_CHILDSUM: return pick<__bf16, 2, K_CS_INT, -1, 2>(nk);
        default: return {};
    }
}
