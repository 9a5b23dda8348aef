// The split tile: fp32 batches of a thousand rows and more on the bf16 matrix
// instructions.
//
// An fp32 value is the sum of three bf16 values to the last bit (8 + 8 + 8
// significant bits), so a fp32 product is nine bf16 products, of which the six
// largest leave out less than 2^-24 of it.  v_mfma_f32_16x16x32_bf16 adds 32
// of them in fp32 in the time of 4 fp32 values' v_mfma_f32_16x16x4_f32: six of
// them take 108 cycles where the fp32 form takes 272.  The weights' pieces are
// made once per forward (split_weights), the operand rows are split here.
//
// Layout: 4 waves share 16 * RB rows; each has 16 units of its own with all
// their gates, so that no weight fragment is read twice in a work-group: they
// go from L2 straight to registers, each gate's for the next chunk of 32 k
// asked for as soon as the gate's products of this one are issued.  The rows'
// pieces are what the waves share: each wave splits its part of the chunk after
// next once and hands it round through the LDS in operand order (16 bytes a
// lane in a row: no bank conflicts).  Bound by the matrix instructions (10,247
// rows of 512 by 1,280: 75 us, 1,075 TFLOP/s of bf16 products, the rate of a
// large bf16 matrix product on this card), and for fewer rows than fill the CUs
// by a work-group's own chain of loads, 27, 15 and 13 us for 64, 32 and 16 rows
// of that size.  Against the fp32 products of the large and streamed tiles, us:
// 10,247 rows 167 and 75, 4,075 rows 53 and 32, 2,019 rows 30 and 19, 790 rows
// 16.5 and 13.6, 30,842 rows of 256 by 768 131 and 75.
//
// Rounding: six products a term into one running total would round it six times
// where an fp32 product rounds it once, which shows where few terms of a row are
// not zero (16 of 512: 2-norm error 1.62e-7 for 1.08e-7).  So the five small
// products add up in accumulators of their own, a 256th of the total's size and
// below its rounding, and the total takes one product a chunk: 16 of 512 0.87e-7,
// one of 512 0.78e-7 for 0.78e-7, dense rows 1.1e-7 for 3.5e-7.  Five gates over 64
// rows have no registers for that: there a chunk's six products are summed from
// zero and join the total by an addition (its kinds read no x; dense 1.0e-7).
// The price is 7% of the large launches (70 to 75 us at 10,247 rows).
#pragma once

#include "cell_kernels.h"

namespace edbk {

// Pieces of the 8 values of a lane's operand fragment, rounded to nearest.  The
// first two stay finite: a value past the largest bf16 one (finfo.min among
// them) takes that as its first piece and leaves the rest to the others, and
// what is not finite goes on to the last piece, whose only product is with the
// weight's first (never zero for a weight that is not).  Products past 2^136 are
// infinite or NaN, where fp32's are infinite.
__device__ __forceinline__ void split8(const uint4& lo, const uint4& hi, uint4 (&o)[3]) {
    typedef float v2f __attribute__((ext_vector_type(2)));
    typedef __bf16 v2bf __attribute__((ext_vector_type(2)));
    constexpr float MOST[2] = {0x1.FEp127f, 0x1p120f};   // of a finite value's first and second piece
#pragma unroll
    for (int i = 0; i < 4; ++i) {
        const uint4& s = i < 2 ? lo : hi;
        v2f v = {__uint_as_float((&s.x)[2 * (i & 1)]), __uint_as_float((&s.x)[2 * (i & 1) + 1])};
#pragma unroll
        for (int k = 0; k < 3; ++k) {
            const v2f r = k == 2 ? v : v2f{__builtin_amdgcn_fmed3f(v.x, -MOST[k & 1], MOST[k & 1]),
                                           __builtin_amdgcn_fmed3f(v.y, -MOST[k & 1], MOST[k & 1])};
            const v2bf b = __builtin_convertvector(r, v2bf);
            const uint32_t u = __builtin_bit_cast(uint32_t, b);
            (&o[k].x)[i] = u;
            if (k == 2) break;
            v.x -= __uint_as_float(u << 16);
            v.y -= __uint_as_float(u & 0xFFFF0000u);
        }
    }
}

// Row blocks of 16 a work-group: 4 (variant 18), 2 (19) or 1 (20, for batches
// that would leave CUs idle).
__host__ __device__ constexpr int split_rb(int sc) { return 4 >> sc; }
constexpr int SPLIT_TU = 64;   // units of a work-group

// One tile: rows [16 RB (tile / nut), + 16 RB) x units [64 (tile % nut), + 64).
template <int KIND, int RB>
__device__ __forceinline__ void split_tile(const BatchArgs& a, int tile) {
    using KT = Kind<KIND>;
    constexpr int G = KT::G, NFX = KT::NFIX, TM = 16 * RB;
    constexpr int NSEG = (KT::X ? 1 : 0) + NFX;
    constexpr int NCR = reads_child_c<KIND>() ? NFX : 0;
    constexpr int KC = 4 / RB;         // chunks of 32 k a step: one row fragment per wave
    // chunks of weights ahead: 16 rows have less matrix time to hide a load's; 32 rows lose by the
    // second set of registers (2,019 rows of 512 by 1,280: 18.9 us for 18.3)
    constexpr int BD = RB == 1 ? 2 : 1;
    // the small products in accumulators of their own (where the registers hold them), else
    // each chunk's products summed before they join the total
    constexpr bool LOW = G * RB <= 16;
    constexpr uint32_t OOB = 0x80000000u;
    static_assert(!KT::RAG && NSEG >= 1 && RB <= 4, "positional kinds");
    __shared__ __align__(16) uint4 rows[2][KC][RB][3][64];
    __shared__ __align__(16) int tab[1 + NCR][TM];   // result rows, then the children's (-1: none)

    // Tile order: unit tiles fastest while an XCD's L2 (4 MB) holds the weights,
    // else row tiles fastest, so that an XCD works on few unit tiles (1,227 rows of
    // 1,024 by 2,560: 47.6 us for 55.4; 1,701 rows of 256 by 768: 11.2 for 10.2)
    const int nub = a.Hu / 16, nut = (nub + 3) / 4, nrt = (a.m + TM - 1) / TM;
    const bool rows_first = a.Hu * a.K * G >= 1 << 19;
    const int rt = rows_first ? tile % nrt : tile / nut, ut = rows_first ? tile / nrt : tile % nut;
    const int row0 = rt * TM;
    const int nrows = min(TM, a.m - row0);
    const int tid = threadIdx.x, lane = tid & 63;
    const int wave = __builtin_amdgcn_readfirstlane(tid >> 6);
    const int ub = ut * 4 + wave;          // past the last block: the wave only splits rows
    const int E = a.E, Ep = a.Ep, H = a.H, Hk = a.Hk, nch = a.K / 32;

    const __amdgpu_buffer_rsrc_t rx = make_rsrc(a.xmat, KT::X ? (uint32_t)a.n_xrows * (uint32_t)E * 4u : 0u);
    const __amdgpu_buffer_rsrc_t rh = make_rsrc(a.arena_h, (uint32_t)a.n_slots * (uint32_t)H * 4u);
    const __amdgpu_buffer_rsrc_t rw = make_rsrc(a.W, (uint32_t)nub * G * nch * 3072u);

    // this wave's row fragment of a step: row block arb, chunk akc of the step
    const int arb = wave % RB, akc = wave / RB;
    const int ar = arb * 16 + (lane & 15);
    uint32_t soff[NSEG];               // byte offset of each segment's source row (OOB: zero)
    {
        const bool ok = ar < nrows;
        int s = 0;
        if constexpr (KT::X) soff[s++] = ok ? (uint32_t)seg_row(a.x, row0 + ar) * (uint32_t)E * 4u : OOB;
#pragma unroll
        for (int p = 0; p < NFX; ++p)
            soff[s++] = !ok ? OOB : a.fix[p].kind == S_NONE ? 0u : (uint32_t)seg_row(a.fix[p], row0 + ar) * (uint32_t)H * 4u;
    }
    for (int i = tid; i < TM * (1 + NCR); i += 256) {
        const int r = i % TM, p = i / TM - 1;
        int v = -1;
        if (r < nrows) {
            if (p < 0) v = seg_row(a.res, row0 + r);
#pragma unroll
            for (int k = 0; k < NCR; ++k)
                if (p == k && a.fix[k].kind != S_NONE) v = seg_row(a.fix[k], row0 + r);
        }
        tab[1 + p][r] = v;
    }

    uint4 ra[2];
    auto load_rows = [&](int step) {
        const int c = step * KC + akc;               // uniform
        int col = c * 32, lim = KT::X ? E : H, end = KT::X ? Ep : Hk;
        uint32_t base = soff[0];
#pragma unroll
        for (int s = 1; s < NSEG; ++s)
            if (col >= end) { col -= end; base = soff[s]; lim = H; end = Hk; }
        const bool xs = KT::X && c * 32 < Ep;
        if (c >= nch) lim = 0;
        col += (lane >> 4) * 8;
#pragma unroll
        for (int i = 0; i < 2; ++i) {
            const uint32_t off = col + 4 * i < lim ? base + (uint32_t)(col + 4 * i) * 4u : OOB;
            ra[i] = __builtin_bit_cast(uint4, xs ? __builtin_amdgcn_raw_buffer_load_b128(rx, off, 0, 0)
                                                 : __builtin_amdgcn_raw_buffer_load_b128(rh, off, 0, 0));
        }
    };
    auto split_rows = [&](int buf) {
        uint4 o[3];
        split8(ra[0], ra[1], o);
#pragma unroll
        for (int k = 0; k < 3; ++k) rows[buf][akc][arb][k][lane] = o[k];
    };
    v8bf b[BD][G][3];
    const int ubl = min(ub, nub - 1);
    auto load_w = [&](int d, int g, int c) {
        // past the last chunk: the last one again, unused (the buffer's bounds check does not
        // hold for a scalar offset past its end)
        const uint32_t base = (uint32_t)((ubl * G + g) * nch + min(c, nch - 1)) * 3072u;
#pragma unroll
        for (int k = 0; k < 3; ++k)
            b[d][g][k] = __builtin_bit_cast(v8bf, __builtin_amdgcn_raw_buffer_load_b128(rw, lane * 16 + k * 1024, base, 0));
    };
    // the LDS exchange alone: loads into registers stay in flight across it
    auto barrier = [&]() {
        asm volatile("s_waitcnt lgkmcnt(0)" ::: "memory");
        __builtin_amdgcn_s_barrier();
        asm volatile("" ::: "memory");
    };

    v4f acc[G][RB], low[LOW ? G : 1][RB];
#pragma unroll
    for (int g = 0; g < G; ++g)
#pragma unroll
        for (int rb = 0; rb < RB; ++rb) acc[g][rb] = low[LOW ? g : 0][rb] = v4f{0.f, 0.f, 0.f, 0.f};

    // smallest first; with sums of their own, in the order that frees the weights for their next load
    constexpr int PA[6] = {LOW ? 0 : 2, LOW ? 1 : 0, LOW ? 0 : 1, LOW ? 2 : 1, LOW ? 1 : 0, 0};
    constexpr int PB[6] = {LOW ? 2 : 0, LOW ? 1 : 2, 1, 0, LOW ? 0 : 1, 0};
    load_rows(0);
#pragma unroll
    for (int d = 0; d < BD; ++d)
#pragma unroll
        for (int g = 0; g < G; ++g) load_w(d, g, d);
    split_rows(0);
    load_rows(1);
    barrier();
    const int steps = (nch + KC - 1) / KC;
    for (int s = 0; s < steps; ++s) {
        const int buf = s & 1;
#pragma unroll
        for (int kc = 0; kc < KC; ++kc) {
            const int c = s * KC + kc;
            if (KC > 1 && c >= nch) break;
            v8bf f[RB][3];
#pragma unroll
            for (int rb = 0; rb < RB; ++rb)
#pragma unroll
                for (int k = 0; k < 3; ++k) f[rb][k] = __builtin_bit_cast(v8bf, rows[buf][kc][rb][k][lane]);
            v4f sums[2][RB];
#pragma unroll
            for (int g = 0; g < G; ++g) {
#pragma unroll
                for (int t = 0; t < 6; ++t)
#pragma unroll
                    for (int rb = 0; rb < RB; ++rb) {
                        v4f& d = !LOW ? sums[g & 1][rb] : t < 5 ? low[g][rb] : acc[g][rb];
                        d = __builtin_amdgcn_mfma_f32_16x16x32_bf16(f[rb][PA[t]], b[kc % BD][g][PB[t]],
                                                                    LOW || t ? d : v4f{0.f, 0.f, 0.f, 0.f}, 0, 0, 0);
                    }
                if (!LOW && g > 0)
#pragma unroll
                    for (int rb = 0; rb < RB; ++rb) acc[g - 1][rb] += sums[(g - 1) & 1][rb];
                if (kc == 0 && g == G - 1) {
                    split_rows(buf ^ 1);   // past the last step: zeros, unused
                    load_rows(s + 2);
                }
                load_w(kc % BD, g, c + BD);
                // keeps the gates apart: left alone, the scheduler sinks every load to the step's end
                __builtin_amdgcn_sched_barrier(0);
            }
            if (!LOW)
#pragma unroll
                for (int rb = 0; rb < RB; ++rb) acc[G - 1][rb] += sums[(G - 1) & 1][rb];
        }
        barrier();
    }
    if (ub >= nub) return;

    // ---- epilogue: every lane holds 4 rows of each block for its unit ----
    const int u = ub * 16 + (lane & 15);
    const __amdgpu_buffer_rsrc_t rc = make_rsrc(a.arena_c, (uint32_t)a.n_slots * (uint32_t)H * 4u);
    float bz[G], cc[NCR > 0 ? NCR : 1][RB][4];
    int res[RB][4];
#pragma unroll
    for (int g = 0; g < G; ++g) bz[g] = a.bias[g * a.Hu + u];
#pragma unroll
    for (int rb = 0; rb < RB; ++rb) {
        const int r = rb * 16 + (lane >> 4) * 4;
#pragma unroll
        for (int i = 0; i < 4; ++i) res[rb][i] = tab[0][r + i];
#pragma unroll
        for (int p = 0; p < NCR; ++p)
#pragma unroll
            for (int i = 0; i < 4; ++i) {
                const int sr = tab[1 + p][r + i];
                const uint32_t off = sr >= 0 ? ((uint32_t)sr * (uint32_t)H + (uint32_t)u) * 4u : OOB;
                cc[p][rb][i] = __uint_as_float(__builtin_amdgcn_raw_buffer_load_b32(rc, off, 0, 0));
            }
    }
    float* const hout = reinterpret_cast<float*>(a.arena_h);
#pragma unroll
    for (int rb = 0; rb < RB; ++rb)
#pragma unroll
        for (int i = 0; i < 4; ++i) {
            float z[G], cp[NFX > 0 ? NFX : 1], c, h;
#pragma unroll
            for (int g = 0; g < G; ++g) z[g] = (LOW ? acc[g][rb][i] + low[g][rb][i] : acc[g][rb][i]) + bz[g];
            cp[0] = 0.f;
#pragma unroll
            for (int p = 0; p < NCR; ++p) cp[p] = cc[p][rb][i];
            cell_update<KIND>(z, cp, 0.f, 0.f, 0, c, h);
            if (res[rb][i] >= 0 && u < H) {
                a.arena_c[(size_t)res[rb][i] * H + u] = c;
                hout[(size_t)res[rb][i] * H + u] = h;
            }
        }
}

// One work-group per tile, in the XCD-aware order of the large tile.
template <int KIND, int SC>
__global__ __launch_bounds__(256, 2) void split_kernel(BatchArgs a) {
    constexpr int TM = 16 * split_rb(SC);
    const int nut = (a.Hu / 16 + 3) / 4;
    const int ntile = ((a.m + TM - 1) / TM) * nut;
    const int per = (ntile + 7) / 8;
    const int tile = (int)(blockIdx.x & 7) * per + (int)(blockIdx.x >> 3);
    if (tile >= ntile) return;
    split_tile<KIND, split_rb(SC)>(a, tile);
}

}  // namespace edbk
