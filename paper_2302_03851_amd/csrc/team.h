// Team launches (team_kernel.h) as the host sees them: the kernels by family,
// and the planning of a schedule's tail into teams.
#pragma once

#include <cstdint>
#include <vector>

#include "edb_internal.h"

namespace edb {

// The combinations of cell types a team launch serves, by what its
// work-groups hold in registers.
enum TeamFamily { TF_CHAIN, TF_NARY, TF_NARY2, TF_GRU, TF_GRID, TF_LATTICE, TF_LGRU, TF_CHILDSUM, TF_COUNT };

struct TeamEntry {
    const void* fn = nullptr;
    int (*lds)(int blk_ints, int rows) = nullptr;   // dynamic LDS bytes
    int nk = 0;                                     // k-groups a wave holds
};

// The kernel of a family for cells of dtype whose reduction has at most
// 8 * nk k-groups, with ub unit blocks a work-group; fn is null if there is none.
TeamEntry team_entry(int family, int dtype, int nk, int ub);
// by source file (one object each)
TeamEntry team_entry_f32(int family, int nk);
TeamEntry team_entry_bf16(int family, int nk, int ub);

struct TeamCell {        // a cell type's sizes
    int kind, G, nfix, nkg;
    bool x, rag;
};

struct TeamPlan {
    int b0 = -1;         // first batch of the launch (-1: no team launch)
    int family = 0, type[2] = {-1, -1}, P = 0, C = 0, ub = 1;
    TeamEntry entry;
    int lds = 0, blk_ints = 0, rows = 0;      // LDS bytes; a team's largest block and row count
    std::vector<int32_t> ints;                // table {offset, ints} per team (relative), then the blocks
    std::vector<int32_t> fill_h, fill_c;      // slots whose h (c) rows start out empty
};

// Decide which tail of the schedule one team launch should run and lay out
// its descriptors.  cost[b]: estimated microseconds of batch b's own launches.
void plan_teams(const edb_graph_t* g, const edb_schedule_t* s, const edb_plan_t* p, const std::vector<TeamCell>& cells,
                int dtype, int hidden, int n_cu, int max_lds, const std::vector<double>& cost, TeamPlan& out);

}  // namespace edb
