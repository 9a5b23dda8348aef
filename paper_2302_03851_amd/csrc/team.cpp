// Planning of a team launch: which tail of the schedule it runs, how the
// instances are dealt to teams, and the descriptors (team_kernel.h).
#include "team.h"

#include <algorithm>
#include <cmath>
#include <cstddef>

namespace edb {
namespace {

constexpr int kTileRows = 16, kTileInts = 8, kRecInts = 8;
constexpr int kMaxChildren = 32, kMaxWords = 16;   // ragged children of a child-sum tile, of a lattice tile
constexpr int kMaxTeam = 32;                       // work-groups of a team

int family_of(int k0, int k1, int dtype) {
    if (k1 < 0) {
        switch (k0) {
            case EDB_CELL_LSTM_CHAIN: return TF_CHAIN;
            // fp32 trees stay on their launches: 16-row fp32 products take a team
            // 2.3 us a tile, which a single mini-batch gains from (64 trees of 256
            // units 101 -> 76 us) and several in flight lose by (55 -> 71 us each)
            case EDB_CELL_NARY_INTERNAL: return dtype == EDB_BF16 ? TF_NARY : -1;
            case EDB_CELL_GRU_INTERNAL: return dtype == EDB_BF16 ? TF_GRU : -1;
            // fp32 grids stay on their launches: their states grow along the grid and
            // carry rounding differences with them, so the order of the sums is kept
            case EDB_CELL_GRID: return dtype == EDB_BF16 ? TF_GRID : -1;
            case EDB_CELL_CS_INTERNAL: return TF_CHILDSUM;
            case EDB_CELL_LAT_CHAR: case EDB_CELL_LAT_WORD: return TF_LATTICE;
            case EDB_CELL_LGRU_EDGE: case EDB_CELL_POOL_MEAN: return TF_LGRU;
            default: return -1;
        }
    }
    const int lo = std::min(k0, k1), hi = std::max(k0, k1);
    if (lo == EDB_CELL_NARY_INTERNAL && hi == EDB_CELL_NARY_INTERNAL) return dtype == EDB_BF16 ? TF_NARY2 : -1;
    if (lo == EDB_CELL_LAT_CHAR && hi == EDB_CELL_LAT_WORD) return TF_LATTICE;
    if (lo == EDB_CELL_LGRU_EDGE && hi == EDB_CELL_POOL_MEAN) return TF_LGRU;
    return -1;
}

// Batches of at most 4 rows per team use the 4-row products (fp32).
bool four_rows(int m, int C, int dtype, int kind) {
    return dtype == EDB_F32 && kind != EDB_CELL_CS_INTERNAL && m <= 4 * C;
}

// Estimated microseconds of one step of `rows` rows of a team of P: per tile
// the exchange between the work-groups and the cell update (longer in larger
// teams), and the matrix-core work (two waves a SIMD; 14, 34 and 18 cycles a
// product).  Measured per tile: chains of 64 units (P 4) 1.1 us, lattices of
// 200 units (P 13) 1.9, bf16 chains of 256 units 2.0, trees of 256 units 2.8
// (4-row form) and 4.2, grids of 256 units 5.3, child-sum cells of 512 units 3.1.
double step_us(const TeamCell& c, int nk, int ub, int P, int dtype, int rows, bool four) {
    if (rows <= 0) return 0.0;
    const int tr = four ? 4 : kTileRows;
    const double tiles = (rows + tr - 1) / tr;
    const double cyc = dtype == EDB_F32 ? (four ? 14.0 : 34.0) * 4 : 18.0;
    const double mma = 2.0 * (c.G + (c.rag ? 1 : 0)) * nk * ub * cyc / 2400.0;
    const double own = 0.6 + 0.075 * P + (c.kind == EDB_CELL_CS_INTERNAL ? 0.8 : 0.0);
    return 0.2 + tiles * (own + mma);
}

constexpr double kFixedUs = 8.0;   // the launch, the weights into registers

}  // namespace

TeamEntry team_entry(int family, int dtype, int nk, int ub) {
    if (dtype == EDB_BF16) return team_entry_bf16(family, nk, ub);
    return ub == 1 ? team_entry_f32(family, nk) : TeamEntry{};
}

void plan_teams(const edb_graph_t* g, const edb_schedule_t* s, const edb_plan_t* p, const std::vector<TeamCell>& cells,
                int dtype, int hidden, int n_cu, int max_lds, const std::vector<double>& cost, TeamPlan& out) {
    out = TeamPlan{};
    const int B = p->B, H = hidden;
    if (B < 2) return;
    const int ub = dtype == EDB_BF16 && H > 256 ? 2 : 1;
    const int P = (H + 16 * ub - 1) / (16 * ub);
    if (P > kMaxTeam || P > n_cu) return;
    auto rows_of = [&](int b) { return s->batch_ptr[b + 1] - s->batch_ptr[b]; };

    // the longest tail of one family's types whose rows fit a tile
    int ty[2] = {-1, -1}, first = B;
    for (int b = B - 1; b >= 0; --b) {
        const int t = s->batch_type[b];
        int n0 = ty[0], n1 = ty[1];
        if (t != n0 && t != n1) {
            if (n0 < 0) n0 = t;
            else if (n1 < 0) n1 = t;
            else break;
            if (family_of(cells[n0].kind, n1 < 0 ? -1 : cells[n1].kind, dtype) < 0) break;
        }
        const TeamCell& c = cells[t];
        bool fits = true;
        if (c.kind == EDB_CELL_CS_INTERNAL || c.kind == EDB_CELL_LAT_CHAR) {
            const int most = c.kind == EDB_CELL_CS_INTERNAL ? kMaxChildren : kMaxWords;
            for (int i = s->batch_ptr[b]; i < s->batch_ptr[b + 1] && fits; ++i) {
                const int32_t v = p->order[i];
                int n = 0;
                for (int64_t k = g->child_ptr[v] + c.nfix; k < g->child_ptr[v + 1]; ++k) n += g->child_idx[k] >= 0;
                fits = n <= most;
            }
        }
        if (c.kind == EDB_CELL_LAT_CHAR || c.kind == EDB_CELL_LAT_WORD) {
            // Work-groups exchange a character's h and a word's c, nothing else: a word as
            // a positional child or a character as a ragged one keeps its batch apart.
            for (int i = s->batch_ptr[b]; i < s->batch_ptr[b + 1] && fits; ++i) {
                const int64_t k0 = g->child_ptr[p->order[i]];
                for (int64_t k = k0; k < g->child_ptr[p->order[i] + 1] && fits; ++k) {
                    const int32_t ch = g->child_idx[k];
                    fits = ch < 0 || cells[g->op_type[ch]].kind != (k < k0 + c.nfix ? EDB_CELL_LAT_WORD : EDB_CELL_LAT_CHAR);
                }
            }
        }
        if (!fits) break;
        ty[0] = n0;
        ty[1] = n1;
        first = b;
    }
    if (first > B - 2) return;
    // which type takes which slot of the family's kernel
    const int fam = family_of(cells[ty[0]].kind, ty[1] < 0 ? -1 : cells[ty[1]].kind, dtype);
    const int second_kind = fam == TF_LATTICE ? EDB_CELL_LAT_WORD : fam == TF_LGRU ? EDB_CELL_POOL_MEAN : -1;
    if (second_kind >= 0) {
        if (cells[ty[0]].kind == second_kind) std::swap(ty[0], ty[1]);
    } else if (fam == TF_NARY2 && ty[0] > ty[1]) {
        std::swap(ty[0], ty[1]);
    }
    int nkg = 0;
    for (int i = 0; i < 2; ++i)
        if (ty[i] >= 0) nkg = std::max(nkg, cells[ty[i]].nkg);
    const int nk = (nkg + 7) / 8;
    const TeamEntry en = team_entry(fam, dtype, nk, ub);
    if (!en.fn) return;

    // the tail of least estimated time, for C teams
    std::vector<double> before(B + 1, 0.0);
    for (int b = 0; b < B; ++b) before[b + 1] = before[b] + cost[b];
    auto best_tail = [&](int C) {
        double tail = kFixedUs, best = before[B];
        int b0 = B;
        int64_t N = 0, kids = 0, tiles = 0;   // a team's share, a tenth to spare for uneven components
        for (int b = B - 1; b >= first; --b) {
            const TeamCell& c = cells[s->batch_type[b]];
            const int m = rows_of(b);
            N += m;
            if (c.rag) kids += p->ragged_pool[p->ragged_off[b] + m];
            tiles += 1 + (m + C - 1) / C / 4;
            const int64_t R = N * 11 / (10 * C) + 8;
            if (en.lds((int)(4 + kTileInts * tiles + kRecInts * R + 2 * (kids * 11 / (10 * C) + 8)), (int)R) > max_lds) break;
            tail += step_us(c, en.nk, ub, P, dtype, (m + C - 1) / C, four_rows(m, C, dtype, c.kind));
            if (before[b] + tail < best) {
                best = before[b] + tail;
                b0 = b;
            }
        }
        return b0;
    };
    int C = n_cu / P, b0 = best_tail(C);
    if (b0 > B - 2) return;

    // connected components of the tail: union-find over its nodes, every root
    // the smallest of its component (scratch kept per thread)
    const int n0 = s->batch_ptr[b0], N = s->batch_ptr[B] - n0;
    static thread_local std::vector<int32_t> at, work;
    if ((int)at.size() < g->V) at.resize(g->V, -1);   // node -> place in the tail; -1 between calls
    work.resize((size_t)4 * N);
    int32_t *up = work.data(), *comp = up + N, *local = comp + N, *sorted = local + N;
    const int32_t* order = p->order.data() + n0;
    const int64_t* cptr = g->child_ptr.data();
    const int32_t* cidx = g->child_idx.data();
    struct Clear {   // whatever way this function is left
        std::vector<int32_t>& v;
        const int32_t* o;
        int n;
        ~Clear() {
            for (int i = 0; i < n; ++i) v[o[i]] = -1;
        }
    } clear{at, order, N};
    auto find = [&](int32_t i) {
        while (up[i] != i) {
            up[i] = up[up[i]];
            i = up[i];
        }
        return i;
    };
    int64_t n_kids = 0;
    for (int i = 0; i < N; ++i) {   // batch order: a row's children come before it
        const int32_t v = order[i];
        at[v] = i;
        int32_t mine = i;
        up[i] = i;
        n_kids += cptr[v + 1] - cptr[v];
        for (int64_t k = cptr[v]; k < cptr[v + 1]; ++k) {
            const int32_t c = cidx[k] < 0 ? -1 : at[cidx[k]];
            if (c < 0) continue;
            const int32_t r = find(c);
            if (r < mine) {
                up[mine] = r;
                mine = r;
            } else if (r > mine) {
                up[r] = mine;
            }
        }
    }
    std::vector<int32_t> size;
    for (int i = 0; i < N; ++i) {
        const int32_t r = find(i);
        if (r == i) {
            comp[i] = (int32_t)size.size();
            size.push_back(0);
        } else {
            comp[i] = comp[r];
        }
        ++size[comp[i]];
    }
    if ((int)size.size() < C) {   // fewer teams than planned for: is the tail still worth it?
        C = (int)size.size();
        if (best_tail(C) > b0) return;
    }
    // largest component first, to the team with the fewest rows
    std::vector<int32_t> by(size.size()), team_of(size.size());
    for (size_t i = 0; i < by.size(); ++i) by[i] = (int32_t)i;
    std::stable_sort(by.begin(), by.end(), [&](int32_t a, int32_t b) { return size[a] > size[b]; });
    std::vector<std::pair<int64_t, int>> load(C);
    for (int c = 0; c < C; ++c) load[c] = {0, c};
    auto more = [](const std::pair<int64_t, int>& a, const std::pair<int64_t, int>& b) { return a > b; };
    std::make_heap(load.begin(), load.end(), more);
    for (int32_t c : by) {
        std::pop_heap(load.begin(), load.end(), more);
        load.back().first += size[c];
        team_of[c] = load.back().second;
        std::push_heap(load.begin(), load.end(), more);
    }
    // the teams' rows in batch order
    std::vector<int32_t> first_row(C + 1, 0);
    for (int i = 0; i < N; ++i) {
        comp[i] = team_of[comp[i]];
        local[i] = first_row[comp[i] + 1]++;
    }
    for (int c = 0; c < C; ++c) first_row[c + 1] += first_row[c];
    for (int i = 0; i < N; ++i) sorted[first_row[comp[i]] + local[i]] = i;

    double worst = 0.0;
    std::vector<int32_t>& ints = out.ints;
    ints.reserve((size_t)2 * C + 16 + (size_t)kRecInts * N + (size_t)kTileInts * (N / 4 + (size_t)C * (B - b0)) + 2 * (size_t)n_kids);
    ints.assign((size_t)2 * C, 0);
    std::vector<int32_t> tiles, kids;
    for (int c = 0; c < C; ++c) {
        const int32_t* R = sorted + first_row[c];
        const int n_rows = first_row[c + 1] - first_row[c];
        // the tiles: rows of one batch, as many as a tile holds
        tiles.clear();
        double us = kFixedUs;
        int b = b0, n_kids_team = 0;
        for (int i = 0; i < n_rows;) {
            while (R[i] + n0 >= s->batch_ptr[b + 1]) ++b;
            const int last = s->batch_ptr[b + 1] - n0;
            int end = i;
            while (end < n_rows && R[end] < last) ++end;
            const int t = s->batch_type[b];
            const TeamCell& cell = cells[t];
            const bool four = four_rows(rows_of(b), C, dtype, cell.kind);
            const int tr = four ? 4 : kTileRows;
            const int most = cell.kind == EDB_CELL_CS_INTERNAL ? kMaxChildren
                             : cell.kind == EDB_CELL_LAT_CHAR ? kMaxWords : 1 << 30;
            us += step_us(cell, en.nk, ub, P, dtype, end - i, four);
            const size_t tiles0 = tiles.size();
            while (i < end) {
                const int row0 = i;
                int nch = 0, chm = 0;
                if (!cell.rag) {
                    i = std::min(end, i + tr);
                } else {
                    for (; i < end && i - row0 < tr; ++i) {
                        const int32_t v = order[R[i]];
                        int nr = 0;
                        for (int64_t k = cptr[v] + cell.nfix; k < cptr[v + 1]; ++k) nr += cidx[k] >= 0;
                        if (i > row0 && nch + nr > most) break;
                        nch += nr;
                        chm = std::max(chm, nr);
                    }
                }
                const int32_t h[kTileInts] = {t == ty[0] ? 0 : 1, i - row0, row0, n_kids_team, nch, chm, four, 0};
                tiles.insert(tiles.end(), h, h + kTileInts);
                n_kids_team += nch;
            }
            for (size_t k = tiles0; k < tiles.size(); k += kTileInts) tiles[k + 7] = (int32_t)((tiles.size() - k) / kTileInts);
        }
        worst = std::max(worst, us);
        // the block: head, tiles, row records, child list
        const size_t off = (ints.size() + 3) / 4 * 4;
        const size_t n_ints = (4 + tiles.size() + (size_t)n_rows * kRecInts + 2 * (size_t)n_kids_team + 3) / 4 * 4;
        ints.resize(off + n_ints);
        int32_t* q = ints.data() + off;
        const int32_t head[4] = {(int32_t)(tiles.size() / kTileInts), n_rows, n_kids_team, 0};
        q = std::copy(head, head + 4, q);
        q = std::copy(tiles.begin(), tiles.end(), q);
        int32_t* kids = q + (size_t)n_rows * kRecInts;
        int nk = 0;
        for (size_t k = 0; k < tiles.size(); k += kTileInts) {
            const TeamCell& cell = cells[ty[tiles[k]]];
            for (int i = tiles[k + 2]; i < tiles[k + 2] + tiles[k + 1]; ++i, q += kRecInts) {
                const int32_t v = order[R[i]];
                const int64_t k0 = cptr[v];
                q[0] = p->slot[v];
                q[1] = cell.x ? g->x_row[v] : -1;
                q[2] = q[3] = 0;
                q[4] = q[5] = -1;
                for (int f = 0; f < cell.nfix; ++f) {
                    const int32_t ch = cidx[k0 + f];
                    if (ch < 0) continue;   // absent: the zero row
                    q[2 + f] = p->slot[ch];
                    if (at[ch] >= 0) q[4 + f] = local[at[ch]];
                }
                q[6] = nk;
                if (cell.rag)
                    for (int64_t e = k0 + cell.nfix; e < cptr[v + 1]; ++e) {
                        const int32_t ch = cidx[e];
                        if (ch < 0) continue;
                        kids[2 * nk] = p->slot[ch];
                        kids[2 * nk + 1] = at[ch] < 0 ? -1 : local[at[ch]];
                        ++nk;
                    }
                q[7] = nk;
            }
        }
        ints[2 * c] = (int32_t)off;
        ints[2 * c + 1] = (int32_t)n_ints;
        out.blk_ints = std::max(out.blk_ints, (int)n_ints);
        out.rows = std::max(out.rows, n_rows);
    }
    out.lds = en.lds(out.blk_ints, out.rows);
    // the rows of a team must fit its LDS, and the busiest team must still beat the launches
    if (out.lds > max_lds || worst >= before[B] - before[b0]) {
        out = TeamPlan{};
        return;
    }
    out.fill_h.reserve(N);
    for (int b = b0; b < B; ++b) {
        std::vector<int32_t>& f = cells[s->batch_type[b]].kind == EDB_CELL_LAT_WORD ? out.fill_c : out.fill_h;
        for (int i = s->batch_ptr[b]; i < s->batch_ptr[b + 1]; ++i) f.push_back(p->slot[p->order[i]]);
    }
    out.b0 = b0;
    out.family = fam;
    out.type[0] = ty[0];
    out.type[1] = ty[1];
    out.P = P;
    out.C = C;
    out.ub = ub;
    out.entry = en;
}

}  // namespace edb
