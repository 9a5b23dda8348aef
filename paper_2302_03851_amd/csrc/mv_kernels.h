// MV-RNN (Table 2): the matrix-vector products of a vector batch.
//
// An MV-RNN node with left child (a, A) and right child (b, B) computes its
// vector from [B a ; A b].  A child's d x d matrix lives in the arena as d
// rows, row j = column j of the matrix, so B a = sum_j a_j * (row j of B) is
// a weighted sum of arena rows.  The vector batch's descriptors give, per
// node, its two vector children (positional lists 0 and 1) and a ragged list
// of exactly 2d entries: the d column rows of A, then the d column rows of B.
// mv_matvec_kernel writes u[r] = [B a, A b] (2d values of T per row); the
// batch's GEMM then reads u as its x operand.  mv_vec_kernel does both in one
// launch.
#pragma once

#include <hip/hip_runtime.h>

#include "cell_kernels.h"

namespace edbk {

// Grid: ceil(2 m / 4) work-groups of 4 waves; wave w handles row w / 2, half
// w % 2 (0: B a, 1: A b).  fp32 rows: lane l = 16 g + q loads 16 bytes
// (columns 4q .. 4q+3 of a 64-column block) of weighted row j = 4 i + g, so
// one wave instruction reads four rows; each lane group g accumulates its
// rows in order, and the four groups' sums are added at the end (g 0 + g 1,
// then + (g 2 + g 3)).  H is a multiple of 4 (16-byte rows).
template <typename T>
__global__ __launch_bounds__(256) void mv_matvec_kernel(BatchArgs a, T* __restrict__ u) {
    static_assert(sizeof(T) == 4, "fp32 rows");
    const int w = blockIdx.x * 4 + (threadIdx.x >> 6), lane = threadIdx.x & 63;
    if (w >= 2 * a.m) return;
    const int r = w >> 1, half = w & 1, H = a.H;
    const int grp = lane >> 4, q = lane & 15;
    const float* h = reinterpret_cast<const float*>(a.arena_h);
    // half 0: B a (weights: the left vector, rows: the right matrix's columns)
    const int vrow = seg_row(half == 0 ? a.fix[0] : a.fix[1], r);
    const int e0 = a.rag_ptr[r] + (half == 0 ? H : 0);
    const float* vec = h + (size_t)vrow * H;
    float* out = reinterpret_cast<float*>(u) + (size_t)r * 2 * H + (size_t)half * H;
    for (int c0 = 0; c0 < H; c0 += 64) {
        const int c = c0 + 4 * q;
        const int cc = c < H ? c : H - 4;   // lanes past H read a valid chunk, store nothing
        float4 acc = make_float4(0.f, 0.f, 0.f, 0.f);
        int j = grp;
        for (; j + 4 < H; j += 8) {   // rows j and j + 4 of this lane group
            const int m0 = seg_row(a.rag, e0 + j), m1 = seg_row(a.rag, e0 + j + 4);
            const float w0 = vec[j], w1 = vec[j + 4];
            const float4 v0 = *reinterpret_cast<const float4*>(h + (size_t)m0 * H + cc);
            const float4 v1 = *reinterpret_cast<const float4*>(h + (size_t)m1 * H + cc);
            acc.x = fmaf(w0, v0.x, acc.x); acc.y = fmaf(w0, v0.y, acc.y);
            acc.z = fmaf(w0, v0.z, acc.z); acc.w = fmaf(w0, v0.w, acc.w);
            acc.x = fmaf(w1, v1.x, acc.x); acc.y = fmaf(w1, v1.y, acc.y);
            acc.z = fmaf(w1, v1.z, acc.z); acc.w = fmaf(w1, v1.w, acc.w);
        }
        for (; j < H; j += 4) {
            const int m0 = seg_row(a.rag, e0 + j);
            const float w0 = vec[j];
            const float4 v0 = *reinterpret_cast<const float4*>(h + (size_t)m0 * H + cc);
            acc.x = fmaf(w0, v0.x, acc.x); acc.y = fmaf(w0, v0.y, acc.y);
            acc.z = fmaf(w0, v0.z, acc.z); acc.w = fmaf(w0, v0.w, acc.w);
        }
        // sum over the four lane groups: (g0 + g1) + (g2 + g3)
        acc.x += __shfl_xor(acc.x, 16); acc.y += __shfl_xor(acc.y, 16);
        acc.z += __shfl_xor(acc.z, 16); acc.w += __shfl_xor(acc.w, 16);
        acc.x += __shfl_xor(acc.x, 32); acc.y += __shfl_xor(acc.y, 32);
        acc.z += __shfl_xor(acc.z, 32); acc.w += __shfl_xor(acc.w, 32);
        if (grp == 0 && c < H) *reinterpret_cast<float4*>(out + c) = acc;
    }
}

// A whole vector batch for d <= 64: grid of (m + 1) / 2 work-groups of 4 waves,
// two rows each.  A wave's matrix-vector product is mv_matvec_kernel's (wave w:
// row w / 2, half w % 2; the same sums in the same order) with all of its 64
// row loads in flight (their numbers come by one load, lane to lane: loaded one
// by one, each waits for the last, and a launch takes 7 us); then wave w multiplies both rows by the w-th quarter of
// the reduction's weights (lane = unit, weights read 16 bytes of k at a time,
// asked for before the matrices), and the quarters are added in order.  Bound by
// its chain of loads (list, matrix rows), which two launches went through with a
// launch's own 4 us each: 564 rows 10.3 us in two and 7.1 in one, 116 rows 10.0
// and 5.1, 2 rows 8.8 and 4.0, and at 5,119 rows, where the matrices' bytes
// bound both, 54 and 47.  Wider cells keep the two launches, whose tiles reuse the weights.
constexpr int MV_MAX_H = 64;
__global__ __launch_bounds__(256) void mv_vec_kernel(BatchArgs a) {
    constexpr int NI = MV_MAX_H / 4, NW = 2 * MV_MAX_H / 16;   // matrix rows a lane group, weight loads a lane
    __shared__ __align__(16) float u[2][2 * MV_MAX_H];
    __shared__ float part[4][2][MV_MAX_H];
    const int lane = threadIdx.x & 63, wave = threadIdx.x >> 6;
    const int H = a.H, K = a.K, nq = K / 4;      // the weights' 16-byte pieces of k per unit
    const float* h = reinterpret_cast<const float*>(a.arena_h);
    // weights: piece f = wave * per + i of unit `lane` (packed [unit block][K / 16][64 lanes][16 bytes])
    const int per = (nq + 3) / 4;
    float4 wv[NW];
#pragma unroll
    for (int i = 0; i < NW; ++i) {
        const int f = wave * per + i;
        wv[i] = make_float4(0.f, 0.f, 0.f, 0.f);
        if (i < per && f < nq)
            wv[i] = reinterpret_cast<const float4*>(a.W)[((lane >> 4) * (K / 16) + (f >> 2)) * 64 + (f & 3) * 16 + (lane & 15)];
    }
    {
        const int r = blockIdx.x * 2 + (wave >> 1), half = wave & 1;
        const int grp = lane >> 4, q = lane & 15, c = 4 * q;
        float4 acc = make_float4(0.f, 0.f, 0.f, 0.f);
        if (r < a.m) {
            const int vrow = seg_row(half == 0 ? a.fix[0] : a.fix[1], r);
            const int e0 = a.rag_ptr[r] + (half == 0 ? H : 0);
            const float* vec = h + (size_t)vrow * H;
            const int cc = c < H ? c : H - 4;   // lanes past H read a valid chunk, store nothing
            // lane j holds row j and its weight: one load each, then from lane to lane
            const int jl = min(lane, H - 1);
            const int my_row = seg_row(a.rag, e0 + jl);
            const float my_wt = vec[jl];
            float4 v[NI];
#pragma unroll
            for (int i = 0; i < NI; ++i)
                v[i] = *reinterpret_cast<const float4*>(h + (size_t)__shfl(my_row, 4 * i + grp) * H + cc);
#pragma unroll
            for (int i = 0; i < NI; ++i) {
                const float wt = __shfl(my_wt, 4 * i + grp);
                if (4 * i + grp >= H) continue;
                acc.x = fmaf(wt, v[i].x, acc.x); acc.y = fmaf(wt, v[i].y, acc.y);
                acc.z = fmaf(wt, v[i].z, acc.z); acc.w = fmaf(wt, v[i].w, acc.w);
            }
        }
        acc.x += __shfl_xor(acc.x, 16); acc.y += __shfl_xor(acc.y, 16);
        acc.z += __shfl_xor(acc.z, 16); acc.w += __shfl_xor(acc.w, 16);
        acc.x += __shfl_xor(acc.x, 32); acc.y += __shfl_xor(acc.y, 32);
        acc.z += __shfl_xor(acc.z, 32); acc.w += __shfl_xor(acc.w, 32);
        if (grp == 0 && c < H) *reinterpret_cast<float4*>(&u[wave >> 1][half * H + c]) = acc;
        const int pad = 2 * H + lane;           // the reduction's padding
        if (half == 1 && pad < K) u[wave >> 1][pad] = 0.f;
    }
    __syncthreads();
    float z[2] = {0.f, 0.f};
#pragma unroll
    for (int i = 0; i < NW; ++i) {
        const int f = wave * per + i;
        if (i >= per || f >= nq) continue;
#pragma unroll
        for (int r = 0; r < 2; ++r) {
            const float4 x = *reinterpret_cast<const float4*>(&u[r][4 * f]);
            z[r] = fmaf(x.x, wv[i].x, z[r]); z[r] = fmaf(x.y, wv[i].y, z[r]);
            z[r] = fmaf(x.z, wv[i].z, z[r]); z[r] = fmaf(x.w, wv[i].w, z[r]);
        }
    }
    part[wave][0][lane] = z[0];
    part[wave][1][lane] = z[1];
    __syncthreads();
    const int r = blockIdx.x * 2 + wave;
    if (wave >= 2 || r >= a.m || lane >= H) return;
    float zz[1] = {((part[0][wave][lane] + part[1][wave][lane]) + part[2][wave][lane]) + part[3][wave][lane] + a.bias[lane]};
    float cp[1] = {0.f}, cn, hn;
    cell_update<K_MV_VEC>(zz, cp, 0.f, 0.f, 0, cn, hn);
    const size_t at = (size_t)seg_row(a.res, r) * H + lane;
    a.arena_c[at] = cn;
    reinterpret_cast<float*>(a.arena_h)[at] = hn;
}

}  // namespace edbk
