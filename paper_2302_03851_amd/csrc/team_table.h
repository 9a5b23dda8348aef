// Choice among the instances of a family's team kernel (device files only).
#pragma once

#include "team.h"
#include "team_kernel.h"

// The instance with the fewest k-groups a wave that still holds nk (NKS ascending).
template <typename T, int UB, int K0, int K1, int NK, int... NKS>
edb::TeamEntry pick(int nk) {
    if (nk <= NK)
        return {reinterpret_cast<const void*>(&edbk::team_kernel<T, NK, UB, K0, K1>),
                [](int blk_ints, int rows) { return edbk::TeamLds<T, NK, UB, K0, K1>::bytes(blk_ints, rows); }, NK};
    if constexpr (sizeof...(NKS) > 0) return pick<T, UB, K0, K1, NKS...>(nk);
    else return {};
}
