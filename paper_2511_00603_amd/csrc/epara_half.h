// Half panels of libepara: the panel tiles of a launch (epara_panel.h), each multiplied by two workgroups that share a
// compute unit, 128 of its 256 rows apiece.
//
// A panel tile has a unit to itself, one wave per SIMD, so nothing hides its start and its epilogue.  Where K is short (a vision
// transformer's K = 768) they are a third of the time.  Here a workgroup of four waves takes 128 rows x 256 columns (gated:
// 128 hidden columns) with at most 256 registers a wave, and two of them share a unit: while one waits for its first operands,
// finishes or stores, the other one multiplies.  The waves split the half by columns as in a panel tile (wave w: two fragments
// of 32 columns; gated: gate and up of the same 32 hidden columns), weights go straight into registers (a ring of two pairs of
// K stages), activations through a ring of four LDS buffers of one pair each.  A fragment of activations read from the LDS
// feeds two products (a block tile's, epara_block_tile.h: one), half of what the LDS can deliver at the matrix cores' rate.
// Sums run over K in the same order and with the same instructions as in a panel tile: the same bits.
//
// What bounds it: the K loop runs at the rate the power limit leaves (1.4 PFLOP/s bf16, matrix cores 73 % busy at 1.64 GHz), as a panel tile's
// does; of the rest, 18 us of 72 for 768 tiles of K = 768 are left of a panel tile's 27 (GELU: 27 of 81 and 47 of 101).  FFN-up of eight
// ViT-B/16 services (14775 rows, 768 -> 3072, GELU): 102 -> 87 us; 8192 x 1024 -> 4096, GELU: 79.5 -> 68.3.  Starting the second workgroup of a
// unit 1 .. 14 us later, or giving one of the two priority, makes it slower (88 .. 91 us): they drift apart by themselves.
#ifndef EPARA_HALF_H
#define EPARA_HALF_H

#include "epara_device.h"

namespace {

constexpr int HALF_ROWS = 128, HALF_RING = 4;
constexpr int HALF_BIAS_LDS_OFFSET = HALF_RING * HALF_ROWS * 128;       // the ring (64 KiB); the epilogue parks the outputs in the same place
constexpr int HALF_LDS_BYTES = HALF_BIAS_LDS_OFFSET + 1024;             // and the bias of the tile's 256 columns

// A visit of a workgroup's list, looked up while the visit before waits for its first operands.
struct half_visit { int slot; epara_tile tl; };

// The next visit of list `list` at or after slot s whose panel tile has rows in this half; slot >= n_slots: none.
__device__ __forceinline__ void half_next(half_visit& v, const epara_group_args* __restrict__ args, const epara_tile* __restrict__ tiles,
                                          const int32_t* __restrict__ order, int s, int n_slots, int stride, int m_half)
{
    for (; s < n_slots; s += stride) {
        asm volatile("" : "+s"(s));                              // indexed from the table's start, so that the load stays a scalar one
        const int t = order[s];
        if (t < 0) continue;
        v.tl = tiles[order_tile(t)];
        if (v.tl.cls < N_STREAM_CLASSES || v.tl.rows <= m_half) continue;
        asm volatile("" :: "s"(args[v.tl.group].K), "s"(args[v.tl.group].scale));      // into the scalar cache
        break;
    }
    v.slot = s;
}

// FM: fragments of 32 rows that hold rows of the batch.
template <int DT, bool GATED, int FM>
__device__ __forceinline__ void half_tile(const half_visit& v, int m_half, int out_dtype, char* lds, half_visit& next,
                                          const epara_group_args* __restrict__ args, const epara_tile* __restrict__ tiles,
                                          const int32_t* __restrict__ order, int n_slots, int stride)
{
    static_assert(DT == EPARA_BF16, "bf16 only");
    constexpr int ESZ = 2, EPC = 16 / ESZ, KF = 4 * EPC;         // elements per 16-byte chunk, per stage
    constexpr int SLOT = FM * 4096;                              // bytes of a pair: FM x 32 rows x 128 bytes
    int tid = threadIdx.x;
    asm volatile("" : "+v"(tid));                                // what is derived from it is computed per tile
    const int lane = tid & 63;
    const int wave = __builtin_amdgcn_readfirstlane(tid >> 6);
    const int r32 = lane & 31, h = lane >> 5;
    ldsptr l3 = (ldsptr)lds;
    const epara_group_args& ga = args[v.tl.group];
    const int K = ga.K, N = ga.N, m0 = v.tl.m0 + m_half, n0 = v.tl.n0, rows = min(v.tl.rows - m_half, HALF_ROWS), cols = v.tl.cols;
    const int KSP = ((K + KF - 1) / KF + 3) & ~3, n_pairs = KSP >> 1;

    // ---- activations: instruction j of a pair covers rows 8 (4 j + wave) .. + 7; lane l writes chunk l % 8 of row l / 8
    // and fetches the chunk that belongs there (chunk ^ (row / 2) % 8: fragment reads are free of bank conflicts)
    const __amdgpu_buffer_rsrc_t xrsrc = __builtin_amdgcn_make_buffer_rsrc(
        const_cast<char*>(static_cast<const char*>(ga.X)) + static_cast<size_t>(m0) * K * ESZ, 0, -1, 0x00020000);
    const int x_chunk = (lane & 7) ^ ((4 * (wave & 1) + (lane >> 4)) & 7);
    const uint32_t pitch = static_cast<uint32_t>(K * ESZ);
    auto x_at = [&](int row) { return static_cast<uint32_t>(min(row, rows - 1)) * pitch + static_cast<uint32_t>(x_chunk * 16); };
    // only the last fragment has rows past the batch
    const uint32_t x_first = x_at(8 * wave + (lane >> 3)), x_last = x_at(8 * (4 * (FM - 1) + wave) + (lane >> 3));
    // Chunks past K come from chunk 0 (the weights are zero there).
    auto x_issue = [&](int p, int j) {
        const int left = K - p * 2 * KF;                         // elements of K from this pair on
        uint32_t off = j == FM - 1 ? x_last : x_first;
        off -= x_chunk * EPC >= left ? static_cast<uint32_t>(x_chunk * 16) : 0u;
        const int so = (left > 0 ? p * 128 : 0) + (j < FM - 1 ? j * 32 * static_cast<int>(pitch) : 0);
        __builtin_amdgcn_raw_ptr_buffer_load_lds(xrsrc, (__attribute__((address_space(3))) void*)(l3 + (p & (HALF_RING - 1)) * SLOT + (4 * j + wave) * 1024),
                                                 16, off, so, 0, 0);
    };
    // ---- weights: fragment fn of the wave is two packed column blocks side by side; lane (r32, h) takes chunk 2 s2 + h of
    // column r32 % 16 of block r32 / 16
    const int NB = (N + 15) >> 4;
    const int nb0 = min((n0 >> 4) + (GATED ? 2 : 4) * wave, NB - 1);
    __amdgpu_buffer_rsrc_t wrsrc[2];
    uint32_t w_off[2];
#pragma unroll
    for (int fn = 0; fn < 2; ++fn) {
        const int rel = min((GATED ? 0 : 2 * fn) + (r32 >> 4), NB - 1 - nb0);      // a block past N only feeds columns that are not stored
        w_off[fn] = static_cast<uint32_t>(rel) * static_cast<uint32_t>(KSP) * 1024u + static_cast<uint32_t>((h * 16 + (r32 & 15)) * 16);
        const void* base = (GATED && fn == 1) ? ga.W2 : ga.W;
        wrsrc[fn] = __builtin_amdgcn_make_buffer_rsrc(const_cast<char*>(static_cast<const char*>(base)) +
                                                      static_cast<size_t>(nb0) * KSP * 1024, 0, -1, 0x00020000);
    }
    v4i w[2][4][2];                                              // [pair % 2][quarter of its K][fn]
    auto w_issue = [&](int p, int fn, int i) -> v4i {
        return __builtin_amdgcn_raw_buffer_load_b128(wrsrc[fn], w_off[fn] + i * 512, p * 2048, 0);
    };
    v16f acc[2][FM];
#pragma unroll
    for (int fn = 0; fn < 2; ++fn)
#pragma unroll
        for (int fm = 0; fm < FM; ++fm)
#pragma unroll
            for (int e = 0; e < 16; ++e) acc[fn][fm][e] = 0.f;
    constexpr int SETS = FM == 4 ? 1 : 2;
    v4i xf[SETS][FM];
    const int sw = (r32 >> 1) & 7;
    const ldsptr xbase = l3 + r32 * 128;
    uint32_t xf_off[4];
#pragma unroll
    for (int i = 0; i < 4; ++i) xf_off[i] = static_cast<uint32_t>(((2 * i + h) ^ sw) << 4);
    auto frag = [&](int p, int i, int fm) -> v4i { return *reinterpret_cast<lds_v4i>(xbase + xf_off[i] + (p & (HALF_RING - 1)) * SLOT + fm * 4096); };

    // ---- one step multiplies a quarter of a pair's K: 2 x FM products.  Under them the fragments of the next step are read
    // (FM = 4: each into the register it has just left, six products ahead of its use; fewer fragments: into a second set), the
    // weight registers are refilled two pairs ahead right after their last use, and the activation loads of the pair two
    // ahead are issued in the first steps.  At most one memory instruction between two products, pinned by the scheduling barriers.
    // The slot of pair p + 2 was last read for pair p - 2, whose products every wave issued before the meeting of pair p - 1.
    // PH: parity of the pair.  MODE: 0 = loads go on; 1 = no loads (the last pair but one); 2 = none and no next pair.
    constexpr int X_STEPS = (FM + 1) / 2;
    auto step = [&](int p, auto ph_tag, auto s_tag, auto mode_tag) {
        constexpr int PH = decltype(ph_tag)::value, S = decltype(s_tag)::value, MODE = decltype(mode_tag)::value;
        constexpr bool LAST = S == 3;
        constexpr int set = S % SETS, nset = (S + 1) % SETS, NS = (S + 1) & 3;
        if constexpr (LAST && MODE < 2) {
            // my part of the next pair has landed: issued after its last activation load were the rest of the pair before and,
            // if loads go on, what this pair has issued in three steps (FM = 1: a weight load may have gone before it)
            wait_vmcnt<2 * (5 - X_STEPS) - (FM == 1 ? 1 : 0) + (MODE == 0 ? 6 + FM : 0)>();
            asm volatile("" ::: "memory");
            __builtin_amdgcn_s_barrier();
            asm volatile("" ::: "memory");
        }
#pragma unroll
        for (int m = 0; m < 2 * FM; ++m) {
            const int fm = m >> 1, fn = m & 1;
            mma32<DT>(acc[fn][fm], w[PH][S][fn], xf[set][fm]);
            if constexpr (!(LAST && MODE == 2)) {
                if (SETS == 1 ? fn == 1 : m < FM) {
                    const int f = SETS == 1 ? fm : m;
                    xf[nset][f] = frag(LAST ? p + 1 : p, NS, f);
                }
            }
            if constexpr (MODE == 0) {
                if (m == 0 && 2 * S < FM) x_issue(p + 2, 2 * S);
                if (m == (FM > 2 ? 3 : 1) && 2 * S + 1 < FM) x_issue(p + 2, 2 * S + 1);
                if (m == 2 * FM - 2) w[PH][S][0] = w_issue(p + 2, 0, S);
                if (m == 2 * FM - 1) w[PH][S][1] = w_issue(p + 2, 1, S);
            }
            __builtin_amdgcn_sched_barrier(0);
        }
    };
    auto pair = [&](int p, auto ph_tag, auto mode_tag) {
        step(p, ph_tag, act_tag<0>{}, mode_tag);
        step(p, ph_tag, act_tag<1>{}, mode_tag);
        step(p, ph_tag, act_tag<2>{}, mode_tag);
        step(p, ph_tag, act_tag<3>{}, mode_tag);
    };

    // ---- the bias of this wave's 64 columns, older than every other load of the tile
    __attribute__((address_space(3))) float* bias3 = (__attribute__((address_space(3))) float*)(l3 + HALF_BIAS_LDS_OFFSET) + wave * 64;
    if constexpr (!GATED) {
        if (ga.bias) {
            const __amdgpu_buffer_rsrc_t brsrc = __builtin_amdgcn_make_buffer_rsrc(const_cast<float*>(ga.bias), 0, -1, 0x00020000);
            __builtin_amdgcn_raw_ptr_buffer_load_lds(brsrc, (__attribute__((address_space(3))) void*)bias3, 4,
                                                     static_cast<uint32_t>(min(n0 + wave * 64 + lane, N - 1)) * 4u, 0, 0, 0);
        } else bias3[lane] = 0.f;
        __builtin_amdgcn_sched_barrier(0);
    }
#pragma unroll
    for (int p = 0; p < 2; ++p) {                                // the first two pairs (n_pairs is even)
#pragma unroll
        for (int j = 0; j < FM; ++j) x_issue(p, j);
        __builtin_amdgcn_sched_barrier(0);                       // the waits count on this order
#pragma unroll
        for (int i = 0; i < 4; ++i)
#pragma unroll
            for (int fn = 0; fn < 2; ++fn) w[p][i][fn] = w_issue(p, fn, i);
        __builtin_amdgcn_sched_barrier(0);
    }
    half_next(next, args, tiles, order, v.slot + stride, n_slots, stride, m_half);      // under the wait for the first operands
    __builtin_amdgcn_sched_barrier(0);
    wait_vmcnt<16 + FM>();
    asm volatile("" ::: "memory");
    __builtin_amdgcn_s_barrier();
    asm volatile("" ::: "memory");
#pragma unroll
    for (int fm = 0; fm < FM; ++fm) xf[0][fm] = frag(0, 0, fm);
    __builtin_amdgcn_sched_barrier(0);
    int p = 0;
    for (; p + 2 < n_pairs; p += 2) {
        pair(p, act_tag<0>{}, act_tag<0>{});
        pair(p + 1, act_tag<1>{}, act_tag<0>{});
    }
    pair(p, act_tag<0>{}, act_tag<1>{});
    pair(p + 1, act_tag<1>{}, act_tag<2>{});

    // ---- epilogue: act / gating in registers (a lane holds columns 32 fn + 8 g + 4 h .. + 3 of its wave's, row fm * 32 + r32),
    // then through the LDS, so that a store instruction covers whole row pieces of 512 bytes (gated: 256).  16-byte chunk c
    // of a row sits at c ^ (row % chunks per row).
    __syncthreads();                                             // the ring has been read
    int group = v.tl.group;
    asm volatile("" : "+s"(group));                              // the arguments are read again instead of held
    const epara_group_args& ge = args[group];
    auto finish = [&](auto act) {
        constexpr int ACT = decltype(act)::value;
        constexpr int BN = GATED ? 128 : 256, NCH = BN * ESZ / 16;
        const float sg = ge.scale, s2g = ge.scale2 * ge.out_inv_scale, inv = ge.out_inv_scale;
#pragma unroll
        for (int fn = 0; fn < (GATED ? 1 : 2); ++fn)
#pragma unroll
            for (int g = 0; g < 4; ++g) {
                const int nl = fn * 32 + 8 * g + 4 * h;          // of this wave's columns
                v4f b4 = {0.f, 0.f, 0.f, 0.f};
                if constexpr (!GATED) b4 = *reinterpret_cast<const __attribute__((address_space(3))) v4f*>(bias3 + nl);
#pragma unroll
                for (int fm = 0; fm < FM; ++fm) {
                    float o[4];
#pragma unroll
                    for (int i = 0; i < 4; ++i) {
                        if constexpr (GATED) o[i] = act_fast<EPARA_ACT_SILU>(sg * acc[0][fm][4 * g + i]) * (s2g * acc[1][fm][4 * g + i]);
                        else                 o[i] = act_fast<ACT>(sg * acc[fn][fm][4 * g + i] + b4[i]) * inv;
                    }
                    const int row = fm * 32 + r32, byte = (wave * (GATED ? 32 : 64) + nl) * ESZ;
                    ldsptr at = l3 + row * (NCH * 16) + (((byte >> 4) ^ (row & (NCH - 1))) << 4) + (byte & 15);
                    typedef float v2f __attribute__((ext_vector_type(2)));
                    typedef __bf16 v2bf __attribute__((ext_vector_type(2)));
                    v2u pk;
                    pk[0] = __builtin_bit_cast(uint32_t, __builtin_convertvector((v2f{o[0], o[1]}), v2bf));
                    pk[1] = __builtin_bit_cast(uint32_t, __builtin_convertvector((v2f{o[2], o[3]}), v2bf));
                    *reinterpret_cast<__attribute__((address_space(3))) v2u*>(at) = pk;
                }
            }
        __syncthreads();
        constexpr int RPI = NT / NCH, EPO = 16 / ESZ;            // rows per pass over the threads, elements per chunk
        const int ch = tid % NCH, col = ch * EPO;
        const bool vec_ok = (static_cast<uint32_t>(N) * ESZ) % 16 == 0 && col + EPO <= cols;
        EPARA_GLOBAL char* y = as_global<char>(ge.Y) + (static_cast<size_t>(m0) * N + n0 + col) * ESZ;
#pragma unroll
        for (int r0 = 0; r0 < FM * 32; r0 += RPI) {
            const int row = r0 + tid / NCH;
            if (row >= rows || col >= cols) continue;
            const v4i q = *reinterpret_cast<lds_v4i>(l3 + row * (NCH * 16) + ((ch ^ (row & (NCH - 1))) << 4));
            EPARA_GLOBAL char* yr = y + static_cast<size_t>(row) * N * ESZ;
            if (vec_ok) *reinterpret_cast<EPARA_GLOBAL v4i*>(yr) = q;
            else {
#pragma unroll
                for (int e = 0; e < EPO; ++e)
                    if (col + e < cols) reinterpret_cast<EPARA_GLOBAL uint16_t*>(yr)[e] = static_cast<uint16_t>(static_cast<uint32_t>(q[e / 2]) >> (16 * (e & 1)));
            }
        }
    };
    if constexpr (GATED) finish(act_tag<EPARA_ACT_SILU>{});
    else                 with_act(ge.act, finish);
    __syncthreads();                                             // the next tile's activations land where the outputs were parked
}

template <int DT, bool GATED>
__global__ __launch_bounds__(NT, 2) void grouped_half_kernel(const epara_group_args* __restrict__ args, const epara_tile* __restrict__ tiles,
                                                             const int32_t* __restrict__ order, int n_slots, int n_lists, int out_dtype)
{
    extern __shared__ __attribute__((aligned(16))) char lds[];
    const int second = blockIdx.x >= static_cast<unsigned>(n_lists), m_half = second * HALF_ROWS;
    half_visit v, next;
    half_next(v, args, tiles, order, blockIdx.x - (second ? n_lists : 0), n_slots, n_lists, m_half);
    while (v.slot < n_slots) {
        const int fm = (min(v.tl.rows - m_half, HALF_ROWS) + 31) >> 5;
        if (fm > 3)       half_tile<DT, GATED, 4>(v, m_half, out_dtype, lds, next, args, tiles, order, n_slots, n_lists);
        else if (fm == 3) half_tile<DT, GATED, 3>(v, m_half, out_dtype, lds, next, args, tiles, order, n_slots, n_lists);
        else if (fm == 2) half_tile<DT, GATED, 2>(v, m_half, out_dtype, lds, next, args, tiles, order, n_slots, n_lists);
        else              half_tile<DT, GATED, 1>(v, m_half, out_dtype, lds, next, args, tiles, order, n_slots, n_lists);
        v = next;
    }
}

template <int DT, bool GATED>
hipError_t enqueue_half(unsigned n_lists, hipStream_t stream, const epara_group_args* args, const epara_tile* tiles,
                        const int32_t* order, long n_slots, int out_dtype)
{
    static const hipError_t attr = hipFuncSetAttribute(reinterpret_cast<const void*>(&grouped_half_kernel<DT, GATED>),
                                                       hipFuncAttributeMaxDynamicSharedMemorySize, HALF_LDS_BYTES);
    if (attr != hipSuccess) return attr;
    hipLaunchKernelGGL((grouped_half_kernel<DT, GATED>), dim3(2 * n_lists), dim3(NT), HALF_LDS_BYTES, stream, args, tiles, order,
                       static_cast<int>(n_slots), static_cast<int>(n_lists), out_dtype);
    return hipGetLastError();
}

}  // namespace

#endif
