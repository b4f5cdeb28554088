// fp32 groups of libepara: fp32 matrix cores, K split over the waves of a workgroup.
#ifndef EPARA_F32_H
#define EPARA_F32_H

#include "epara_device.h"

namespace {

// An fp32 tile belongs to a small model: a handful of workgroups, and what a launch takes is the chain of dependent
// memory latencies in one of them.  So a workgroup has sixteen waves and cuts K into pieces of 16 that are dealt to them
// contiguously (16-row class: sixteen parts of K; 64-row class: eight parts for each half of the rows); a wave asks for
// several pieces at once and the partial tiles are added in a fixed order (see f32_do_tile): the result depends on nothing but the
// operands.  Operands go from memory straight into v_mfma_f32_16x16x4_f32 (products and sums in fp32): lane (i, q) loads
// X[row i][k + 4 q .. + 3] and W[k + 4 q + e][column 4 i .. 4 i + 3] as 16-byte pieces; product e of a piece pairs the k
// = 4 q + e of both, and the four columns of a lane belong to four accumulators, so that a lane ends with 4 rows x 4
// consecutive columns.  Measured, three launches of two MLPs (256-512-512-10, 4 and 16 rows): 38.5 -> 23.7 us a pass; one launch of
// 256 rows, 1024 x 1024, five times: 130 -> 69 us, 4096 rows: 257 -> 129 us (four waves that staged 16 or 64 k at a time through
// the LDS and multiplied on the vector units).
// A chain whose grid does not fit the chip with one such workgroup per unit runs workgroups of eight waves, two per unit, in
// which a wave takes two of the sixteen shares one after the other: the same sums in the same order.
constexpr int F32_WAVES = 16, F32_NT = F32_WAVES * 64, F32_BN = 64, F32_HALF_NT = F32_NT / 2;

// A piece of 16 k: RB blocks of 16 rows x 64 columns of one wave.
template <int RB>
struct f32_piece { v4f x[RB], w[4]; };

struct f32_tile {
    const EPARA_GLOBAL float* X;   // first row of the wave
    const EPARA_GLOBAL float* W;   // first column of the tile
    int K, N, rows, cols;          // rows: of the wave
    bool xv, wv;                   // 16-byte pieces of X / W are aligned
};

template <int RB>
__device__ __forceinline__ void f32_fetch(const f32_tile& t, int k0, int lane, f32_piece<RB>& p)
{
    const int i = lane & 15, k = k0 + 4 * (lane >> 4);
    const bool whole = k0 + 16 <= t.K;                           // the same for all lanes
#pragma unroll
    for (int b = 0; b < RB; ++b) {
        // a row past the batch repeats the last one: it only feeds outputs that are not stored
        const EPARA_GLOBAL float* x = t.X + static_cast<size_t>(min(16 * b + i, t.rows - 1)) * t.K + k;
        if (whole && t.xv) p.x[b] = *reinterpret_cast<const EPARA_GLOBAL v4f*>(x);
        else {
#pragma unroll
            for (int e = 0; e < 4; ++e) p.x[b][e] = k + e < t.K ? x[e] : 0.f;
        }
    }
#pragma unroll
    for (int e = 0; e < 4; ++e) {
        const EPARA_GLOBAL float* w = t.W + static_cast<size_t>(k + e) * t.N + 4 * i;
        p.w[e] = v4f{0.f, 0.f, 0.f, 0.f};
        if (t.wv) { if (k + e < t.K && 4 * i < t.cols) p.w[e] = *reinterpret_cast<const EPARA_GLOBAL v4f*>(w); }
        else {
#pragma unroll
            for (int c = 0; c < 4; ++c) if (k + e < t.K && 4 * i + c < t.cols) p.w[e][c] = w[c];
        }
    }
}

// AHEAD pieces of a wave's part of K are in flight while one is multiplied.
template <int RB, int AHEAD>
__device__ __forceinline__ void f32_multiply(const f32_tile& t, int p0, int p1, int lane, v4f (&acc)[RB][4])
{
    f32_piece<RB> ring[AHEAD + 1];
#pragma unroll
    for (int a = 0; a < AHEAD; ++a)
        if (p0 + a < p1) f32_fetch<RB>(t, 16 * (p0 + a), lane, ring[a]);
    for (int p = p0; p < p1; p += AHEAD + 1) {
#pragma unroll
        for (int a = 0; a < AHEAD + 1; ++a) {
            if (p + a >= p1) break;
            if (p + a + AHEAD < p1) f32_fetch<RB>(t, 16 * (p + a + AHEAD), lane, ring[(a + AHEAD) % (AHEAD + 1)]);
#pragma unroll
            for (int e = 0; e < 4; ++e)
#pragma unroll
                for (int b = 0; b < RB; ++b)
#pragma unroll
                    for (int c = 0; c < 4; ++c)
                        acc[b][c] = __builtin_amdgcn_mfma_f32_16x16x4f32(ring[a].x[b][e], ring[a].w[e][c], acc[b][c], 0, 0, 0);
        }
    }
}

// A tile of RB x 16 x HALVES rows; PARTS = F32_WAVES / HALVES parts of K.  At most 64 KiB of partial sums meet in the LDS at a
// time: with eight parts of 64 rows part s + 4 is added to part s first, then the four sums in the order of s; the sixteen
// parts of a 16-row tile are added in the order of K.  WAVES: of the workgroup, which hold F32_WAVES / WAVES shares each.
template <bool CHAIN, int WAVES, int RB, int HALVES>
__device__ __forceinline__ void f32_do_tile(const epara_group_args& ga, const epara_tile& tl, v4f* lds)
{
    constexpr int PARTS = F32_WAVES / HALVES, ROWS = RB * 16 * HALVES, ROUNDS = F32_WAVES / WAVES;
    constexpr int MEET = 65536 / (ROWS * F32_BN * 4) < PARTS ? 65536 / (ROWS * F32_BN * 4) : PARTS;      // parts that fit the LDS
    static_assert(MEET == PARTS || 2 * MEET == PARTS, "parts meet in one or two steps");
    static_assert(ROUNDS == 1 || ROUNDS == 2, "a wave takes one or two shares");
    const int lane = threadIdx.x & 63;
    const int wave = __builtin_amdgcn_readfirstlane(threadIdx.x >> 6);
    const int half = wave % HALVES;                              // the same for both shares
    const int i = lane & 15, q = lane >> 4;
    const int K = ga.K, N = ga.N, row0 = half * RB * 16;
    const int pieces = (K + 15) >> 4;
    v4f acc[RB][4];
    auto multiply = [&](int part) {                              // contiguous shares of the pieces of K
#pragma unroll
        for (int b = 0; b < RB; ++b)
#pragma unroll
            for (int c = 0; c < 4; ++c) acc[b][c] = v4f{0.f, 0.f, 0.f, 0.f};
        const int p0 = static_cast<int>(static_cast<int64_t>(pieces) * part / PARTS), p1 = static_cast<int>(static_cast<int64_t>(pieces) * (part + 1) / PARTS);
        if (row0 < tl.rows) {
            const f32_tile t = {as_global<float>(ga.X) + static_cast<size_t>(tl.m0 + row0) * K, as_global<float>(ga.W) + tl.n0, K, N,
                                tl.rows - row0, tl.cols, (K & 3) == 0, (N & 3) == 0};
            // (two shares: one piece less ahead, or the kernel needs more than the 128 registers of two workgroups per unit)
            f32_multiply<RB, RB == 1 ? (ROUNDS == 2 ? 2 : 3) : 1>(t, p0, p1, lane, acc);
        }
    };
    // quad (row, column quad) of part s at [s][row][quad]; a lane holds rows 4 q + v of each block, columns 4 i .. 4 i + 3
    auto at = [&](int s, int row, int quad) -> v4f& { return lds[(s * ROWS + row) * 16 + quad]; };
    auto dump = [&](int s) {
#pragma unroll
        for (int b = 0; b < RB; ++b)
#pragma unroll
            for (int v = 0; v < 4; ++v) at(s, row0 + 16 * b + 4 * q + v, i) = v4f{acc[b][0][v], acc[b][1][v], acc[b][2][v], acc[b][3][v]};
    };
    const int part = wave / HALVES;
    if constexpr (ROUNDS == 2) {                                 // the upper share first: its sums wait in the LDS
        multiply(part + PARTS / 2);
        dump(MEET < PARTS ? part : part + PARTS / 2);
    }
    multiply(part);
    if constexpr (MEET < PARTS) {
        if (part >= MEET) dump(part - MEET);
        __syncthreads();
        if (part < MEET) {
#pragma unroll
            for (int b = 0; b < RB; ++b)
#pragma unroll
                for (int v = 0; v < 4; ++v) {
                    const v4f other = at(part, row0 + 16 * b + 4 * q + v, i);
#pragma unroll
                    for (int c = 0; c < 4; ++c) acc[b][c][v] += other[c];
                }
        }
        __syncthreads();
    }
    if (part < MEET) dump(part);
    __syncthreads();
    for (int u = threadIdx.x; u < ROWS * 16; u += WAVES * 64) {
        const int row = u >> 4, col = (u & 15) * 4;
        if (row >= tl.rows || col >= tl.cols) continue;
        v4f sum = at(0, row, u & 15);
#pragma unroll
        for (int s = 1; s < MEET; ++s) sum += at(s, row, u & 15);
        EPARA_GLOBAL float* y = as_global<float>(ga.Y) + static_cast<size_t>(tl.m0 + row) * N + tl.n0 + col;
        const EPARA_GLOBAL float* bias = ga.bias ? as_global<float>(ga.bias) + tl.n0 + col : nullptr;
        const int valid = tl.cols - col;
        with_act(ga.act, [&](auto tag) {
            v4f out;
#pragma unroll
            for (int c = 0; c < 4; ++c) {
                const float b = bias && c < valid ? bias[c] : 0.f;
                out[c] = act_apply<decltype(tag)::value>(ga.scale * sum[c] + b);
            }
            if constexpr (!CHAIN) {
                if (valid >= 4 && (N & 3) == 0) { *reinterpret_cast<EPARA_GLOBAL v4f*>(y) = out; return; }
            }
#pragma unroll
            for (int c = 0; c < 4; ++c) if (c < valid) put<CHAIN>(y + c, out[c]);
        });
    }
    __syncthreads();                                             // the partial tiles are free again
}

// The tables of a small launch into the scalar cache while a workgroup waits for its entry of the order: wave w asks for a word of
// the w-th 64-byte line of each.  The look-ups order -> tile -> arguments, each of which names the next, then cost one trip to
// memory and two to that cache instead of three to memory: three launches of two MLPs (256-512-512-10, 4 and 16 rows) 23.6 -> 22.9 us a pass.
constexpr int F32_WARM_BYTES = F32_WAVES * 64;
__device__ __forceinline__ void f32_warm(const epara_group_args* __restrict__ args, uint32_t args_bytes, const epara_tile* __restrict__ tiles, uint32_t tile_bytes,
                                         const int32_t* __restrict__ order, long n_slots)
{
    const uint32_t at = static_cast<uint32_t>(__builtin_amdgcn_readfirstlane(static_cast<int>(threadIdx.x >> 6))) * 64;
    const int a = *reinterpret_cast<const int*>(reinterpret_cast<const char*>(args) + min(at, args_bytes - 4));
    const int t = *reinterpret_cast<const int*>(reinterpret_cast<const char*>(tiles) + min(at, tile_bytes - 4));
    const int o = blockIdx.x < n_slots ? order[blockIdx.x] : 0;
    asm volatile("" :: "s"(a), "s"(t), "s"(o));
}

template <bool CHAIN, int WAVES>
__device__ __forceinline__ void f32_body(const epara_group_args* __restrict__ args, const epara_tile* __restrict__ tiles,
                                         const int32_t* __restrict__ order, long n_slots, chain_ctx* chain)
{
    __shared__ v4f lds[65536 / 16];
    for (long s = blockIdx.x; s < n_slots; s += gridDim.x) {
        const int t = order[s];
        if (t < 0) continue;
        const epara_tile tl = tiles[t];
        if constexpr (CHAIN) chain_wait(*chain, tl.group);
        const epara_group_args ga = args[tl.group];
        if (tl.cls == 0) f32_do_tile<CHAIN, WAVES, 1, 1>(ga, tl, lds);  // class 0 of the fp32 table: at most 16 rows
        else             f32_do_tile<CHAIN, WAVES, 2, 2>(ga, tl, lds);
        if constexpr (CHAIN) chain_done(*chain, tl.group);
    }
}

}  // namespace

#endif
