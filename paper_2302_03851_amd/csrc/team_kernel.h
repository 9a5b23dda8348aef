// Team launch: the tail of a schedule (its last batches, or all of them) in
// one launch.
//
// One launch per batch costs 4-8 us however few rows the batch has: the
// dispatch, then a chain of dependent round trips to memory from cold caches
// (row indices, operand rows and weights, cell states), about 2 us of it
// matrix-core work at most.  Chains and lattices are nothing but such batches.
// Here the instances of the mini-batch (connected components of the tail) are
// dealt to teams of P work-groups.  Work-group p of a team owns 16*UB hidden
// units: it loads their weights for all gates and the whole reduction into
// registers once, keeps its units' cell states of the team's rows in LDS, and
// then walks the team's rows batch by batch, at most 16 rows (a tile) at a
// time.  Only the h rows travel between the work-groups of a team (and the
// words' cell states of a lattice), through the arena itself: they are stored
// and loaded past the L2s (agent scope), and a row that has not been written
// yet holds a pattern that no stored value has (every bit set; the launch
// before fills it in), so a consumer simply reloads an operand fragment until
// it is there.  No flag, no counter and no barrier between work-groups: one
// exchange between 13-16 work-groups takes 1.3-1.6 us with this, 2.0-2.2 us
// with a flag per work-group behind the rows.
//
// Progress.  A work-group takes its place from a ticket counter when it
// starts, so the members of a team are the next P work-groups that run,
// wherever the hardware placed them, and only the last team started can be
// incomplete.  Its members may hold the CUs its missing ones wait for, between
// them and those of other launches (of other processes too), so they wait for
// the last one a bounded time only: the last member to start sets the team's
// state to full; one whose time is up before sets it to left, and then all but
// the last end without having written anything, which makes room.  The last,
// whenever it starts, finds it so and walks the team's rows alone, unit block
// by unit block (the same results; 32 lattices of 200 units 6.8 ms for 0.17).  A full team's
// members all run, so its waits for rows end; each is bounded all the same:
// past `limit` reloads a wave sets the error words, stops waiting for the rest
// of the launch and goes on.  The host keeps few team launches in flight at
// once, so that the slow way is not met within a process.
//
// Work of a tile: 8 waves split the reduction (k-group kg to wave kg % 8),
// the partial sums meet in LDS, and the threads that take a (row, unit) add
// them in wave order.  Tiles of fp32 batches with few rows per team use
// v_mfma_f32_4x4x1 with 4 rows: the packed weights are its B operand as they
// are, with the four k-quarters of a k-group in four lane groups.  It takes
// 14 cycles for 4 rows where the 16-row form takes 34.  Which form a batch
// uses depends on the batch's size alone, never on how its rows were dealt,
// so a row's result does not depend on its team or its place in a tile.
#pragma once

#include "cell_kernels.h"

namespace edbk {

constexpr int TEAM_NT = 512, TEAM_NW = 8;   // threads and waves of a work-group
constexpr int TEAM_ROWS = 16;               // rows of a tile
constexpr int TEAM_CH = 32;                 // children of a child-sum tile
constexpr int TEAM_WORDS = 16;              // words of a lattice-character tile
constexpr int TEAM_TILE_INTS = 8;           // {type, rows, first row, first child, children, most children, 4-row form, tiles of the batch from here}
constexpr int TEAM_REC_INTS = 8;            // {result slot, x row, child slots, their local rows, ragged range}
constexpr int TEAM_FULL = 1, TEAM_LEFT = 2;    // states of a team
constexpr uint32_t TEAM_EMPTY = 0xFFFFFFFFu;   // a word of a row that is not written yet

struct TeamType {
    const uint4* W;
    const float* bias;
    const uint4* Wr;
    const float* br;
    int E, Ep, Hk, Hu, K;
};

struct TeamArgs {
    TeamType t[2];
    const int* ibuf;     // descriptor ints
    int off_table;       // per team {offset of its block in ibuf, ints of the block}
    int* ticket;         // {ticket, error, state of each team}, zero before the launch
    int* error;          // the host's error word (host memory), or none
    int attend;          // how long members wait for the last one, in ticks of 10 ns (below 0: every team is left)
    int P, C, H, n_slots, n_xrows;
    int blk_ints;        // LDS room for a team's block
    int limit;           // reloads of one wait before it gives up
    const void* x;
    void* arena_h;
    float* arena_c;
};

// A team's block: {tiles, rows, children, 0}, the tiles, the row records
// and the child list ({slot, local row} pairs; local row -1: a row that an
// earlier launch wrote).

// 16-byte load that sees what another work-group stored at agent scope.
__device__ __forceinline__ uint4 bload_agent(__amdgpu_buffer_rsrc_t r, uint32_t off) {
    return __builtin_bit_cast(uint4, __builtin_amdgcn_raw_buffer_load_b128(r, (int)off, 0, 16));
}

template <typename T> __device__ __forceinline__ bool team_full(uint4 v);
template <> __device__ __forceinline__ bool team_full<float>(uint4 v) {
    return v.x != TEAM_EMPTY && v.y != TEAM_EMPTY && v.z != TEAM_EMPTY && v.w != TEAM_EMPTY;
}
template <> __device__ __forceinline__ bool team_full<__bf16>(uint4 v) {
    auto f = [](uint32_t w) { return (w & 0xFFFFu) != 0xFFFFu && (w >> 16) != 0xFFFFu; };
    return f(v.x) && f(v.y) && f(v.z) && f(v.w);
}

// Store a value of a row that other work-groups wait for.  A NaN with the
// empty pattern becomes the canonical NaN.
__device__ __forceinline__ void store_agent(float* p, float v) {
    const uint32_t u = __float_as_uint(v);
    __hip_atomic_store(reinterpret_cast<uint32_t*>(p), u == TEAM_EMPTY ? 0x7FC00000u : u, __ATOMIC_RELAXED,
                       __HIP_MEMORY_SCOPE_AGENT);
}
__device__ __forceinline__ void store_agent(__bf16* p, float v) {
    const __bf16 b = (__bf16)v;
    const uint16_t u = __builtin_bit_cast(uint16_t, b);
    __hip_atomic_store(reinterpret_cast<uint16_t*>(p), u == 0xFFFFu ? (uint16_t)0x7FC0u : u, __ATOMIC_RELAXED,
                       __HIP_MEMORY_SCOPE_AGENT);
}

// One k-group of one 16-unit block: 16 rows, or (fp32) 4 rows whose four
// k-quarters accumulate in four lane groups.
template <typename T, int G, int TR>
__device__ __forceinline__ void team_mma(v4f (&acc)[G], const uint4& a, const uint4 (&b)[G]) {
    if constexpr (sizeof(T) == 4) {
#pragma unroll
        for (int j = 0; j < 4; ++j)
#pragma unroll
            for (int g = 0; g < G; ++g) {
                const float av = __uint_as_float((&a.x)[j]), bv = __uint_as_float((&b[g].x)[j]);
                if constexpr (TR == 4) acc[g] = __builtin_amdgcn_mfma_f32_4x4x1f32(av, bv, acc[g], 0, 0, 0);
                else acc[g] = __builtin_amdgcn_mfma_f32_16x16x4f32(av, bv, acc[g], 0, 0, 0);
            }
    } else {
#pragma unroll
        for (int g = 0; g < G; ++g)
            acc[g] = __builtin_amdgcn_mfma_f32_16x16x32_bf16(__builtin_bit_cast(v8bf, a), __builtin_bit_cast(v8bf, b[g]),
                                                            acc[g], 0, 0, 0);
    }
}

// Sum over the PARTS (1, 2 or 8) neighbouring lanes of an item.
template <int PARTS>
__device__ __forceinline__ float lane_sum(float v) {
    auto dpp = [](float x, auto ctrl) {
        return __uint_as_float((uint32_t)__builtin_amdgcn_update_dpp(0, (int)__float_as_uint(x), decltype(ctrl)::value,
                                                                     0xf, 0xf, true));
    };
    if constexpr (PARTS >= 2) v += dpp(v, std::integral_constant<int, 0xB1>{});    // lane ^ 1
    if constexpr (PARTS >= 8) {
        v += dpp(v, std::integral_constant<int, 0x4E>{});                          // lane ^ 2
        v += dpp(v, std::integral_constant<int, 0x141>{});                         // the other four of eight
    }
    return v;
}

template <int KIND>
__host__ __device__ constexpr int team_gates() { return KIND < 0 ? 0 : Kind<KIND < 0 ? 0 : KIND>::G; }
__host__ __device__ constexpr int cmax_(int a, int b) { return a > b ? a : b; }

// LDS of a work-group in 4-byte words: {places, partial sums, ragged partial
// sums, child fragments, children's cell states, biases}, then the team's
// block and the cell states [rows][TU].
template <typename T, int NK, int UB, int K0, int K1>
struct TeamLds {
    static constexpr int TU = 16 * UB;
    static constexpr int G = cmax_(team_gates<K0>(), team_gates<K1>());
    static constexpr int ZROW = G * TU + 4;                  // conflict-free rows
    static constexpr int ZWAVE = TEAM_ROWS * ZROW + 8;
    static constexpr bool CS = K0 == K_CS_INT;
    static constexpr bool LAT = K0 == K_LAT_CHAR;
    static constexpr int NZ = CS || UB > 1 ? 1 : 2;          // one barrier a tile with two sets of partial sums
    static constexpr int ZR_ROWS = CS ? TEAM_CH : LAT ? TEAM_WORDS : 0;
    static constexpr int ZRWAVE = ZR_ROWS ? ZR_ROWS * TU + 8 : 0;
    static constexpr int PLACE = 0;
    static constexpr int Z = 4;
    static constexpr int ZR = Z + NZ * TEAM_NW * ZWAVE;
    static constexpr int FRAG = (ZR + NZ * TEAM_NW * ZRWAVE + 3) / 4 * 4;
    static constexpr int CCH = FRAG + (CS ? TEAM_NW * NK * (TEAM_CH / 16) * 64 * 4 : 0);
    static constexpr int BIAS = CCH + (CS ? TEAM_CH * TU : 0);
    static constexpr int BLK = (BIAS + 2 * 6 * TU + 3) / 4 * 4;
    static constexpr int bytes(int blk_ints, int rows) { return 4 * (BLK + blk_ints + rows * TU); }
};

template <typename T, int NK, int UB, int K0, int K1>
struct Team {
    using L = TeamLds<T, NK, UB, K0, K1>;
    static constexpr int TU = L::TU, KG = Elem<T>::KG, V = Elem<T>::VEC;
    static constexpr uint32_t ES = sizeof(T), OOB = 0x80000000u;

    const TeamArgs& a;
    float* lds;
    const int* blk;          // the team's block in LDS
    const int* rows;         // its row records and its child list
    const int* kids0;
    float* cst;              // cell states of the team's rows
    int tid, lane, wave, u0;
    bool dead = false;       // this wave has given up waiting

    template <int KIND>
    using Weights = uint4[UB][NK][Kind<KIND>::G];

    // The registers of one type: k-group wave + 8 i in slot i (zero past the end).
    template <int G>
    __device__ __forceinline__ void load_weights(uint4 (&w)[UB][NK][G], const uint4* W, int nkg, int p) const {
#pragma unroll
        for (int ub = 0; ub < UB; ++ub)
#pragma unroll
            for (int i = 0; i < NK; ++i)
#pragma unroll
                for (int g = 0; g < G; ++g) {
                    const int kg = wave + TEAM_NW * i;
                    w[ub][i][g] = kg < nkg && W ? W[(((size_t)(p * UB + ub) * G + g) * nkg + kg) * 64 + lane]
                                                : make_uint4(0, 0, 0, 0);
                }
    }

    // Reload `ld` until `ok` holds on every lane (bounded).
    template <typename LD, typename OK>
    __device__ __forceinline__ void wait(LD ld, OK ok) {
        for (int tries = 0; !__all(ok()); ++tries) {
            if (dead || tries >= a.limit) {
                if (!dead && lane == 0) {
                    __hip_atomic_store(a.ticket + 1, 1, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT);
                    if (a.error) __hip_atomic_store(a.error, 1, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_SYSTEM);
                }
                dead = true;
                break;
            }
            asm volatile("" ::: "memory");   // the loads are not hoisted out of the loop
            ld();
        }
    }

    // The tiles [t0, t0 + cnt) of one batch.  They do not depend on each other:
    // while a 16-row tile's gates are computed the next one's operand loads are
    // already in flight (its registers are free by then).
    template <int KIND, int TR, int G>
    __device__ __forceinline__ void step(int ty, const uint4 (&w)[UB][NK][G], const uint4 (&wr)[UB][NK][1], int t0, int cnt) {
        using KT = Kind<KIND>;
        constexpr int NFX = KT::NFIX;
        constexpr bool HX = KT::X;
        constexpr bool CSI = KIND == K_CS_INT, POOL = KIND == K_POOL_MEAN, CHAR = KIND == K_LAT_CHAR;
        const TeamType& t = a.t[ty];
        const int H = a.H;
        const __amdgpu_buffer_rsrc_t rx = make_rsrc(a.x, HX ? (uint32_t)a.n_xrows * (uint32_t)t.E * ES : 0u);
        const __amdgpu_buffer_rsrc_t rh = make_rsrc(a.arena_h, (uint32_t)a.n_slots * (uint32_t)H * ES);
        const __amdgpu_buffer_rsrc_t rc = make_rsrc(a.arena_c, (uint32_t)a.n_slots * (uint32_t)H * 4u);
        const int nkg = t.K / KG, xkg = HX ? t.Ep / KG : 0, hkg = t.Hk / KG;
        constexpr int PARTS = TEAM_NT / (TR * TU);
        const int part = tid % PARTS, item = tid / PARTS, eu = item % TU, er = item / TU;
        const int j = u0 + eu, q = lane >> 4;
        const float* bias = lds + L::BIAS + ty * 6 * TU;

        // a tile: its header, this thread's item, the operand loads in flight
        constexpr bool SEGS = !CSI && !POOL;      // operands [x | child h ...] by row
        constexpr int NC = CSI ? TEAM_CH / 16 : 1;
        constexpr int WV = sizeof(T) == 4 ? 1 : 2;
        int n, row0, ch0, nch, chm;
        const int* kids;
        int4 ra, rb, ea, eb;                      // records of the lane's operand row and of the thread's item
        bool rok, eok;
        float cpre[NFX > 0 ? NFX : 1], ccg[CSI ? UB : 1];
        uint4 av[NC][NK];
        uint32_t off[NC][NK];
        uint32_t poll = 0;                        // bit p: the row of child (tile of children) p is waited for
        uint4 wv[CHAR ? NK : 1][WV];
        uint32_t woff[CHAR ? NK : 1];
        uint32_t wpoll = 0;

        // the wave's number, opaque for every tile: the k-group arithmetic is a few
        // scalar instructions a tile, kept across tiles it would not fit the registers
        int wq = wave;
        auto isx = [&](int i) { return HX && wq + TEAM_NW * i < xkg; };
        auto ldh = [&] {
#pragma unroll
            for (int c = 0; c < NC; ++c)
                if (!CSI || c * 16 < nch)
#pragma unroll
                    for (int i = 0; i < NK; ++i)
                        if (!isx(i)) av[c][i] = bload_agent(rh, off[c][i]);
        };
        auto ldw = [&] {
            if constexpr (CHAR)
#pragma unroll
                for (int i = 0; i < NK; ++i)
#pragma unroll
                    for (int k = 0; k < WV; ++k) wv[i][k] = bload_agent(rc, woff[i] == OOB ? OOB : woff[i] + 16u * k);
        };
        auto issue = [&](int tile) {
            asm volatile("" : "+s"(wq));
            const int* hdr = blk + 4 + TEAM_TILE_INTS * tile;
            const int4 h0 = *reinterpret_cast<const int4*>(hdr);
            const int2 h1 = *reinterpret_cast<const int2*>(hdr + 4);
            n = __builtin_amdgcn_readfirstlane(h0.y);
            row0 = __builtin_amdgcn_readfirstlane(h0.z);
            ch0 = __builtin_amdgcn_readfirstlane(h0.w);
            nch = __builtin_amdgcn_readfirstlane(h1.x);
            chm = __builtin_amdgcn_readfirstlane(h1.y);
            kids = kids0 + 2 * ch0;
            const int r = TR == 4 ? (lane & 3) : (lane & 15);
            rok = r < n;
            const int* rec = rows + TEAM_REC_INTS * (row0 + (rok ? r : 0));
            ra = *reinterpret_cast<const int4*>(rec);
            rb = *reinterpret_cast<const int4*>(rec + 4);
            const int* erec = rows + TEAM_REC_INTS * (row0 + (er < n ? er : 0));
            ea = *reinterpret_cast<const int4*>(erec);
            eb = *reinterpret_cast<const int4*>(erec + 4);
            eok = er < n && j < H;
            if constexpr (SEGS) {
                poll = rok ? (rb.x >= 0 ? 1u : 0u) | (rb.y >= 0 ? 2u : 0u) : 0u;
#pragma unroll
                for (int i = 0; i < NK; ++i) {
                    const int kg = wq + TEAM_NW * i, kh = kg - xkg;
                    const bool second = NFX > 1 && kh >= hkg;
                    const int col = (isx(i) ? kg : second ? kh - hkg : kh) * KG + q * V;
                    const int slot = second ? ra.w : ra.z;
                    if (isx(i)) off[0][i] = rok && col < t.E ? ((uint32_t)ra.y * (uint32_t)t.E + (uint32_t)col) * ES : OOB;
                    else off[0][i] = kg < nkg && rok && col < H ? ((uint32_t)slot * (uint32_t)H + (uint32_t)col) * ES : OOB;
                }
                if constexpr (HX)
#pragma unroll
                    for (int i = 0; i < NK; ++i)
                        if (isx(i)) av[0][i] = bload(rx, off[0][i]);
                ldh();
            }
            if constexpr (CHAR) {   // the words' cell states (fp32 rows): row = word
                const int wd = lane & 15;
                const bool wok = wd < nch;
                const int ws = kids[2 * (wok ? wd : 0)], wl = kids[2 * (wok ? wd : 0) + 1];
                wpoll = wok && wl >= 0;
#pragma unroll
                for (int i = 0; i < NK; ++i) {
                    const int kg = wq + TEAM_NW * i, col = kg * KG + q * V;
                    const bool ok = wok && kg < hkg && col < H;
                    woff[i] = ok ? ((uint32_t)ws * (uint32_t)H + (uint32_t)col) * 4u : OOB;
                }
                if (nch > 0) ldw();
            }
            if constexpr (CSI) {   // the children's h rows
                poll = 0;
#pragma unroll
                for (int c = 0; c < NC; ++c) {
                    const int e = c * 16 + (lane & 15);
                    const bool ok = e < nch;
                    const int ks = kids[2 * (ok ? e : 0)], kl = kids[2 * (ok ? e : 0) + 1];
                    poll |= (ok && kl >= 0 ? 1u : 0u) << c;
#pragma unroll
                    for (int i = 0; i < NK; ++i) {
                        const int kg = wq + TEAM_NW * i, col = kg * KG + q * V;
                        const bool use = ok && kg < hkg && col < H;
                        off[c][i] = use ? ((uint32_t)ks * (uint32_t)H + (uint32_t)col) * ES : OOB;
                    }
                }
                ldh();
                // cell states of children that an earlier launch wrote, one (child, unit) a thread
#pragma unroll
                for (int h = 0; h < UB; ++h) {
                    const int e = (tid + TEAM_NT * h) / TU, u = tid % TU;
                    const bool ok = e < nch && u0 + u < H && kids[2 * (e < nch ? e : 0) + 1] < 0;
                    ccg[h] = __uint_as_float(
                        bload32(rc, ok ? ((uint32_t)kids[2 * e] * (uint32_t)H + (uint32_t)(u0 + u)) * 4u : OOB));
                }
            }
            const int ecl[2] = {eb.x, eb.y}, ecs[2] = {ea.z, ea.w};
#pragma unroll
            for (int p = 0; p < NFX; ++p)
                cpre[p] = __uint_as_float(bload32(
                    rc, eok && ecl[p] < 0 ? ((uint32_t)ecs[p] * (uint32_t)H + (uint32_t)j) * 4u : OOB));
        };

        // one tile, its loads issued: the products, the partial sums to LDS, then
        // (with `more`) the next tile's loads, the gates and the stores
        auto body = [&](int tile, auto more) {
            const int zb = L::NZ == 1 ? 0 : tile & 1;
            float* Zr = lds + L::ZR + zb * TEAM_NW * L::ZRWAVE + wave * L::ZRWAVE;
            v4f acc[UB][G];
#pragma unroll
            for (int ub = 0; ub < UB; ++ub)
#pragma unroll
                for (int g = 0; g < G; ++g) acc[ub][g] = v4f{0.f, 0.f, 0.f, 0.f};

            if constexpr (SEGS) {
                // x's products go ahead of the wait for the children
                if constexpr (HX)
#pragma unroll
                    for (int i = 0; i < NK; ++i)
                        if (isx(i))
#pragma unroll
                            for (int ub = 0; ub < UB; ++ub) team_mma<T, G, TR>(acc[ub], av[0][i], w[ub][i]);
                wait(ldh, [&] {
                    bool ok = true;
#pragma unroll
                    for (int i = 0; i < NK; ++i)
                        if (!isx(i)) ok = ok && (!(poll & (NFX > 1 && wq + TEAM_NW * i - xkg >= hkg ? 2u : 1u)) || team_full<T>(av[0][i]));
                    return ok;
                });
#pragma unroll
                for (int i = 0; i < NK; ++i)
                    if (!isx(i) && wq + TEAM_NW * i < nkg)
#pragma unroll
                        for (int ub = 0; ub < UB; ++ub) team_mma<T, G, TR>(acc[ub], av[0][i], w[ub][i]);
                if constexpr (CHAR) {
                    if (nch > 0) {   // the words' link-gate products
                        wait(ldw, [&] {
                            bool ok = true;
#pragma unroll
                            for (int i = 0; i < NK; ++i)
#pragma unroll
                                for (int k = 0; k < WV; ++k) ok = ok && (!wpoll || team_full<float>(wv[i][k]));
                            return ok;
                        });
                        v4f aw[UB][1];
#pragma unroll
                        for (int ub = 0; ub < UB; ++ub) aw[ub][0] = v4f{0.f, 0.f, 0.f, 0.f};
#pragma unroll
                        for (int i = 0; i < NK; ++i)
                            if (wq + TEAM_NW * i < hkg) {
                                uint4 f = wv[i][0];
                                if constexpr (sizeof(T) == 2) {
                                    T* pf = reinterpret_cast<T*>(&f);
                                    const float* ps = reinterpret_cast<const float*>(&wv[i][0]);
#pragma unroll
                                    for (int k = 0; k < V; ++k) pf[k] = from_f<T>(ps[k]);
                                }
#pragma unroll
                                for (int ub = 0; ub < UB; ++ub) team_mma<T, 1, 16>(aw[ub], f, wr[ub][i]);
                            }
#pragma unroll
                        for (int ub = 0; ub < UB; ++ub)
#pragma unroll
                            for (int k = 0; k < 4; ++k) Zr[(q * 4 + k) * TU + ub * 16 + (lane & 15)] = aw[ub][0][k];
                    }
                }
            } else if constexpr (CSI) {
                // the children's forget products, then the child sums from LDS (each
                // wave reads back its own k-groups only)
                wait(ldh, [&] {
                    bool ok = true;
#pragma unroll
                    for (int c = 0; c < NC; ++c)
                        if (c * 16 < nch)
#pragma unroll
                            for (int i = 0; i < NK; ++i) ok = ok && (!(poll >> c & 1u) || team_full<T>(av[c][i]));
                    return ok;
                });
                uint4* fr = reinterpret_cast<uint4*>(lds + L::FRAG) + wave * NK * NC * 64;
#pragma unroll
                for (int c = 0; c < NC; ++c)
                    if (c * 16 < nch) {
#pragma unroll
                        for (int i = 0; i < NK; ++i) fr[(i * NC + c) * 64 + lane] = av[c][i];
                        v4f af[UB][1];
#pragma unroll
                        for (int ub = 0; ub < UB; ++ub) {
                            af[ub][0] = v4f{0.f, 0.f, 0.f, 0.f};
#pragma unroll
                            for (int i = 0; i < NK; ++i) team_mma<T, 1, 16>(af[ub], av[c][i], wr[ub][i]);
#pragma unroll
                            for (int k = 0; k < 4; ++k)
                                Zr[(c * 16 + q * 4 + k) * TU + ub * 16 + (lane & 15)] = af[ub][0][k];
                        }
                    }
#pragma unroll
                for (int h = 0; h < UB; ++h)
                    if ((tid + TEAM_NT * h) / TU < nch) lds[L::CCH + tid + TEAM_NT * h] = ccg[h];
                const int e0 = rok ? rb.z - ch0 : 0, e1 = rok ? rb.w - ch0 : 0;
                float s[NK][V];
#pragma unroll
                for (int i = 0; i < NK; ++i)
#pragma unroll
                    for (int k = 0; k < V; ++k) s[i][k] = 0.f;
                for (int c = 0; c < chm; ++c) {
                    const int e = min(e0 + c, TEAM_CH - 1);
#pragma unroll
                    for (int i = 0; i < NK; ++i) {
                        const uint4 f = fr[(i * NC + (e >> 4)) * 64 + q * 16 + (e & 15)];
                        const T* pf = reinterpret_cast<const T*>(&f);
                        if (e0 + c < e1)
#pragma unroll
                            for (int k = 0; k < V; ++k) s[i][k] += to_f(pf[k]);
                    }
                }
#pragma unroll
                for (int i = 0; i < NK; ++i) {
                    uint4 f;
                    T* pf = reinterpret_cast<T*>(&f);
#pragma unroll
                    for (int k = 0; k < V; ++k) pf[k] = from_f<T>(s[i][k]);
#pragma unroll
                    for (int ub = 0; ub < UB; ++ub) team_mma<T, G, TR>(acc[ub], f, w[ub][i]);
                }
            } else {
                // pooling: the sum of the children's h rows, four children at a time
                const int e0 = rok ? rb.z - ch0 : 0, e1 = rok ? rb.w - ch0 : 0;
                constexpr int CB = 4;
                float s[NK][V];
#pragma unroll
                for (int i = 0; i < NK; ++i)
#pragma unroll
                    for (int k = 0; k < V; ++k) s[i][k] = 0.f;
                uint32_t cb[NK];   // byte offset of the lane's columns in a row
#pragma unroll
                for (int i = 0; i < NK; ++i) {
                    const int kg = wq + TEAM_NW * i, col = kg * KG + q * V;
                    cb[i] = kg < hkg && col < H ? (uint32_t)col * ES : OOB;
                }
                for (int c = 0; c < chm; c += CB) {
                    uint4 pv[CB][NK];
                    uint32_t pr[CB], pp = 0;
#pragma unroll
                    for (int b = 0; b < CB; ++b) {
                        const bool ok = e0 + c + b < e1;
                        const int e = ok ? e0 + c + b : 0;
                        const int ks = kids[2 * e], kl = kids[2 * e + 1];
                        pp |= (ok && kl >= 0 ? 1u : 0u) << b;
                        pr[b] = ok ? (uint32_t)ks * (uint32_t)H * ES : OOB;
                    }
                    auto ldp = [&] {   // past the last child and past H: out of range, zero
#pragma unroll
                        for (int b = 0; b < CB; ++b)
#pragma unroll
                            for (int i = 0; i < NK; ++i)
                                pv[b][i] = bload_agent(rh, __builtin_elementwise_add_sat(pr[b], cb[i]));
                    };
                    ldp();
                    wait(ldp, [&] {
                        bool ok = true;
#pragma unroll
                        for (int b = 0; b < CB; ++b)
#pragma unroll
                            for (int i = 0; i < NK; ++i) ok = ok && (!(pp >> b & 1u) || team_full<T>(pv[b][i]));
                        return ok;
                    });
#pragma unroll
                    for (int b = 0; b < CB; ++b)
#pragma unroll
                        for (int i = 0; i < NK; ++i) {
                            const T* pf = reinterpret_cast<const T*>(&pv[b][i]);
#pragma unroll
                            for (int k = 0; k < V; ++k) s[i][k] += to_f(pf[k]);
                        }
                }
#pragma unroll
                for (int i = 0; i < NK; ++i) {
                    uint4 f;
                    T* pf = reinterpret_cast<T*>(&f);
#pragma unroll
                    for (int k = 0; k < V; ++k) pf[k] = from_f<T>(s[i][k]);
#pragma unroll
                    for (int ub = 0; ub < UB; ++ub) team_mma<T, G, TR>(acc[ub], f, w[ub][i]);
                }
            }

            // every load has returned: said here, where it costs nothing, or the
            // compiler would wait for the stores too before it reuses the registers
#pragma unroll
            for (int c = 0; c < NC; ++c)
#pragma unroll
                for (int i = 0; i < NK; ++i)
                    if constexpr (!POOL) asm volatile("" ::"v"(av[c][i].x));
            if constexpr (CHAR)
#pragma unroll
                for (int i = 0; i < NK; ++i) asm volatile("" ::"v"(wv[i][WV - 1].x));
#pragma unroll
            for (int p = 0; p < NFX; ++p) asm volatile("" ::"v"(cpre[p]));

            // ---- partial sums to LDS (4-row form: row = k-quarter * 4 + row) ----
            float* Zb = lds + L::Z + zb * TEAM_NW * L::ZWAVE;
#pragma unroll
            for (int ub = 0; ub < UB; ++ub)
#pragma unroll
                for (int g = 0; g < G; ++g)
#pragma unroll
                    for (int k = 0; k < 4; ++k)
                        Zb[wave * L::ZWAVE + (q * 4 + k) * L::ZROW + g * TU + ub * 16 + (lane & 15)] = acc[ub][g][k];
            __syncthreads();

            // this tile's item, before the next tile's loads take the registers
            const int ern = n, errow = row0 + er, ech0 = ch0;
            const int4 ia = ea, ib = eb;
            const bool iok = eok;
            const int* ikids = kids;
            float cp[NFX > 0 ? NFX : 1] = {0.f};
            const int ecl[2] = {ib.x, ib.y};
#pragma unroll
            for (int p = 0; p < NFX; ++p) {
                const float cl = cst[(ecl[p] < 0 ? 0 : ecl[p]) * TU + eu];
                cp[p] = ecl[p] < 0 ? cpre[p] : cl;
            }
            if constexpr (decltype(more)::value) issue(tile + 1);

            // ---- gate pre-activations and cell update of this thread's item ----
            float z[G];
            constexpr int WP = TEAM_NW / PARTS;   // waves whose partial sums a lane adds
#pragma unroll
            for (int g = 0; g < G; ++g) {
                float s = 0.f;
#pragma unroll
                for (int v = 0; v < WP; ++v) {
                    const float* zp = Zb + (part * WP + v) * L::ZWAVE + g * TU + eu;
                    if constexpr (TR == 4) {
#pragma unroll
                        for (int k = 0; k < 4; ++k) s += zp[(k * 4 + er) * L::ZROW];
                    } else {
                        s += zp[er * L::ZROW];
                    }
                }
                s = lane_sum<PARTS>(s);
                z[g] = POOL ? s : s + bias[g * TU + eu];
            }
            float racc = 0.f, rden = 0.f;
            int nw = 0;
            if constexpr (POOL) racc = bias[eu];
            if constexpr (CSI || CHAR || POOL) nw = er < ern ? ib.w - ib.z : 0;
            if constexpr (CSI || CHAR) {
                const float* Zrb = lds + L::ZR + zb * TEAM_NW * L::ZRWAVE;
                const float brj = bias[5 * TU + eu];
                for (int c = 0; c < nw; ++c) {
                    const int e = ib.z - ech0 + c;
                    float s = 0.f;
#pragma unroll
                    for (int v = 0; v < WP; ++v) s += Zrb[(part * WP + v) * L::ZRWAVE + e * TU + eu];
                    s = lane_sum<PARTS>(s) + brj;
                    const int kl = ikids[2 * e + 1];
                    float cw;
                    if constexpr (CSI) cw = kl < 0 ? lds[L::CCH + e * TU + eu] : cst[kl * TU + eu];
                    else cw = kl < 0 ? __uint_as_float(bload32(rc, iok ? ((uint32_t)ikids[2 * e] * (uint32_t)H + (uint32_t)j) * 4u : OOB))
                                     : cst[kl * TU + eu];
                    if constexpr (CSI) {
                        racc += sigm(s) * cw;
                    } else {
                        const float ek = __expf(sigm(z[4] + s));
                        racc = fmaf(ek, cw, racc);
                        rden += ek;
                    }
                }
            }
            if (iok && part == 0) {
                float c, h;
                cell_update<KIND>(z, cp, racc, rden, nw, c, h);
                cst[errow * TU + eu] = c;
                const size_t o = (size_t)ia.x * H + j;
                T* hp = reinterpret_cast<T*>(a.arena_h) + o;
                if constexpr (KIND == K_LAT_WORD) {   // its cell state travels, its h is zero
                    store_agent(a.arena_c + o, c);
                    *hp = from_f<T>(h);
                } else {
                    store_agent(hp, h);
                    a.arena_c[o] = c;
                }
            }
            if constexpr (L::NZ == 1) __syncthreads();
        };
        // The last tile's code has no loads behind it: with loads possibly in
        // flight at the end of a batch, the compiler waits for everything (the
        // stores too, about 0.5 us) before the next batch's first load.  Short
        // batches (the 4-row form, pooling) keep one copy of the code.
        if constexpr (TR == 4 || POOL) {
            for (int tile = t0; tile < t0 + cnt; ++tile) {
                issue(tile);
                body(tile, std::false_type{});
            }
        } else {
            issue(t0);
            for (int tile = t0; tile + 1 < t0 + cnt; ++tile) body(tile, std::true_type{});
            body(t0 + cnt - 1, std::false_type{});
        }
    }

    template <int KIND>
    __device__ __forceinline__ void load_bias(const TeamType& t, int ty) {
        constexpr int G = Kind<KIND>::G;
        float* b = lds + L::BIAS + ty * 6 * TU;
        for (int i = tid; i < G * TU; i += TEAM_NT) b[i] = t.bias[(i / TU) * t.Hu + u0 + i % TU];
        if constexpr (Kind<KIND>::RAG)
            for (int i = tid; i < TU; i += TEAM_NT) b[5 * TU + i] = t.br[u0 + i];
    }
};

// The team's state as the member at place p leaves its start: full, or left.
// `seen`: what the last member found in its place.
__device__ __forceinline__ int team_attend(int* state, int seen, bool last, int ticks) {
    auto swap = [&](int to) {
        int was = 0;
        __hip_atomic_compare_exchange_strong(state, &was, to, __ATOMIC_RELAXED, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT);
        return was;
    };
    if (last) return seen || ticks < 0 ? TEAM_LEFT : TEAM_FULL;
    const uint64_t end = wall_clock64() + (uint64_t)ticks;
    for (;;) {
        int now = __hip_atomic_load(state, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT);
        if (!now && wall_clock64() >= end) {
            now = swap(TEAM_LEFT);
            if (!now) now = TEAM_LEFT;
        }
        if (now) return now;
        __builtin_amdgcn_s_sleep(1);
    }
}

// What a work-group of a team does, in LDS whose block of descriptors is loaded:
// the weights of its units in registers, and the walk over the tiles.
template <typename T, int NK, int UB, int K0, int K1>
struct Walker {
    using TM = Team<T, NK, UB, K0, K1>;
    static constexpr int G0 = Kind<K0>::G, G1 = K1 < 0 ? 1 : Kind<K1 < 0 ? 0 : K1>::G;
    TM tm;
    uint4 w0[UB][NK][G0], w1[UB][NK][G1], wr[UB][NK][1];

    __device__ __forceinline__ Walker(const TeamArgs& a, float* lds, int tid)
        : tm{a, lds, nullptr, nullptr, nullptr, lds + TM::L::BLK + a.blk_ints, tid, tid & 63,
             __builtin_amdgcn_readfirstlane(tid >> 6), 0} {
        tm.blk = reinterpret_cast<const int*>(lds + TM::L::BLK);
    }
    // unit block p: its weights to registers, its biases to the LDS
    __device__ __forceinline__ void load(int p) {
        const TeamArgs& a = tm.a;
        tm.u0 = p * TM::TU;
        tm.load_weights(w0, a.t[0].W, a.t[0].K / TM::KG, p);
        if constexpr (K1 >= 0) tm.load_weights(w1, a.t[1].W, a.t[1].K / TM::KG, p);
        if constexpr (Kind<K0>::RAG) tm.load_weights(wr, a.t[0].Wr, a.t[0].Hk / TM::KG, p);
        if (a.t[0].W) tm.template load_bias<K0>(a.t[0], 0);
        if constexpr (K1 >= 0)
            if (a.t[1].W) tm.template load_bias<K1>(a.t[1], 1);
    }
    // the block of descriptors has arrived; returns its number of tiles
    __device__ __forceinline__ int ready() {
        const int nt = __builtin_amdgcn_readfirstlane(tm.blk[0]);
        tm.rows = tm.blk + 4 + TEAM_TILE_INTS * nt;
        tm.kids0 = tm.rows + TEAM_REC_INTS * __builtin_amdgcn_readfirstlane(tm.blk[1]);
        return nt;
    }
    __device__ __forceinline__ void walk(int t, int t1) {
        while (t < t1) {
            const int* hdr = tm.blk + 4 + TEAM_TILE_INTS * t;
            const int ty = __builtin_amdgcn_readfirstlane(hdr[0]), cnt = __builtin_amdgcn_readfirstlane(hdr[7]);
            const bool four = sizeof(T) == 4 && K0 != K_CS_INT && __builtin_amdgcn_readfirstlane(hdr[6]) != 0;
            const int t0 = t;
            t += cnt;
            if (K1 < 0 || ty == 0) {
                if constexpr (sizeof(T) == 4 && K0 != K_CS_INT) {
                    if (four) {
                        tm.template step<K0, 4>(0, w0, wr, t0, cnt);
                        continue;
                    }
                }
                tm.template step<K0, 16>(0, w0, wr, t0, cnt);
            } else if constexpr (K1 >= 0) {
                if constexpr (sizeof(T) == 4) {
                    if (four) {
                        tm.template step<K1, 4>(1, w1, wr, t0, cnt);
                        continue;
                    }
                }
                tm.template step<K1, 16>(1, w1, wr, t0, cnt);
            }
        }
    }
};

template <typename T, int NK, int UB, int K0, int K1>
__global__ __launch_bounds__(TEAM_NT, 2) void team_kernel(TeamArgs a) {
    extern __shared__ __align__(16) float tsmem[];
    using TM = Team<T, NK, UB, K0, K1>;
    using L = typename TM::L;
    int* place = reinterpret_cast<int*>(tsmem);
    if (threadIdx.x == 0) place[0] = __hip_atomic_fetch_add(a.ticket, 1, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT);
    __syncthreads();
    const int id = __builtin_amdgcn_readfirstlane(place[0]);
    const int team = id / a.P, p = id - team * a.P;
    if (team >= a.C) return;
    const bool last = p == a.P - 1;
    int* state = a.ticket + 2 + team;
    int seen = 0;
    if (threadIdx.x == 0 && last)
        __hip_atomic_compare_exchange_strong(state, &seen, a.attend < 0 ? TEAM_LEFT : TEAM_FULL, __ATOMIC_RELAXED, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT);
    int* blk = reinterpret_cast<int*>(tsmem + L::BLK);
    Walker<T, NK, UB, K0, K1> w(a, tsmem, (int)threadIdx.x);
    w.load(p);
    const int boff = a.ibuf[a.off_table + 2 * team], bn = a.ibuf[a.off_table + 2 * team + 1];
    for (int i = threadIdx.x; i < bn / 4; i += TEAM_NT)
        reinterpret_cast<int4*>(blk)[i] = reinterpret_cast<const int4*>(a.ibuf + boff)[i];
    if (threadIdx.x == 0) place[1] = team_attend(state, seen, last, a.attend);
    __syncthreads();
    if (__builtin_amdgcn_readfirstlane(place[1]) != TEAM_LEFT) {
        const int nt = w.ready();
        w.walk(0, nt);
        return;
    }
    if (!last) return;
    // The last member of a team that the others left: every step (the tiles of a batch)
    // with each unit block in turn.  No row is waited for, and the cell states are read
    // back from the arena.  All of it is made anew for each block from values the
    // compiler cannot see through: in one loop with the members' walk, or with
    // anything kept from block to block, it takes registers there (lattices of 200
    // units 176 us and 190) or scratch memory (0.5 us a forward even where unused).
    const int nt = w.ready();
    {
        int* rows = const_cast<int*>(w.tm.rows);
        int* kids = const_cast<int*>(w.tm.kids0);
        for (int i = threadIdx.x; i < blk[1]; i += TEAM_NT) rows[TEAM_REC_INTS * i + 4] = rows[TEAM_REC_INTS * i + 5] = -1;
        for (int i = threadIdx.x; i < blk[2]; i += TEAM_NT) kids[2 * i + 1] = -1;
    }
    for (int t = 0; t < nt;) {
        const int cnt = __builtin_amdgcn_readfirstlane(blk[4 + TEAM_TILE_INTS * t + 7]);
        for (int q = p; q >= 0; --q) {
            __threadfence();    // the blocks before have stored their rows and are done with the LDS
            __syncthreads();
            using Args = const __constant__ TeamArgs;
            Args* ka = (Args*)__builtin_amdgcn_kernarg_segment_ptr();
            int tid = threadIdx.x;
            asm volatile("" : "+s"(ka));
            asm volatile("" : "+v"(tid));
            auto type = [&](int i) {
                return TeamType{ka->t[i].W, ka->t[i].bias, ka->t[i].Wr, ka->t[i].br, ka->t[i].E, ka->t[i].Ep, ka->t[i].Hk, ka->t[i].Hu, ka->t[i].K};
            };
            const TeamArgs b{{type(0), type(1)}, ka->ibuf, ka->off_table, ka->ticket, ka->error, ka->attend, ka->P, ka->C, ka->H, ka->n_slots,
                             ka->n_xrows, ka->blk_ints, ka->limit, ka->x, ka->arena_h, ka->arena_c};
            Walker<T, NK, UB, K0, K1> one(b, tsmem, tid);
            one.ready();
            one.load(q);
            __syncthreads();
            one.walk(t, t + cnt);
        }
        t += cnt;
    }
}

}  // namespace edbk
