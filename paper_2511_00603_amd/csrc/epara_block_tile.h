// Block tiles of libepara: 128 rows x 128 columns of one group (gated groups: 64 hidden columns, i.e. 64 gate +
// 64 up weight columns), two workgroups per compute unit.
//
// A quarter of a panel tile (epara_panel.h), for launches whose panel tiles do not fill the chip or leave a nearly
// empty last round: batches of some hundred rows, a long batch next to tiny ones, a few images.  The four waves
// split the tile by columns as in a panel tile (wave w: all rows of columns 32 w .. 32 w + 31; gated: hidden columns
// 16 w .. 16 w + 15, the lower half of its fragment from the gate matrix, the upper half from the up matrix, so that
// a lane ends with the gate and the up sum of the same outputs), weights go straight into registers, activations
// through a ring of four LDS buffers of one "pair" (two 64-byte K stages) each.  Only the fragments of 32 rows that
// hold rows of the batch are loaded and multiplied (FM = 1 .. 4), so a batch of a few rows costs little more than
// its weight stream.
//
// Two workgroups share a unit (64 KiB of LDS, at most 256 registers each), so nothing is pipelined across tiles:
// while one workgroup waits for its first operands or stores, the other one multiplies.  Sums run over K in the
// same order and with the same instructions as in a panel tile: the results agree bit for bit.
//
// Weights of a group of a single row tile are read by one workgroup once.  In large launches (`once`, by the size of the launch; see weights_once in
// epara_launch.hip) that is done with the non-temporal hint: three SwiGLU services of 75 rows, 4096 -> 11008, 120.6 -> 112.0 us, of 120 rows
// 134.4 -> 128.6, four of 96 rows, 11008 -> 4096, 77.3 -> 69.8.  Where several row tiles share them the hint costs (75 + 130 + 237 rows, a pass
// 236 -> 262 us), and so it does on activations (291).
#ifndef EPARA_BLOCK_TILE_H
#define EPARA_BLOCK_TILE_H

#include "epara_device.h"

namespace {

constexpr int BLOCK_RING = 4;                                    // pairs in flight or being read
constexpr int BLOCK_LDS_BYTES = BLOCK_RING * 128 * 128;          // 64 KiB; the epilogue parks the tile's outputs in the same place

// Split block tiles: three of them per slot of the panel tiles' workspace (four parts of 64 KiB each).  They count in
// front of all partial sums like every other split tile, eight tiles to a counter: partial sums never land on the counters of
// a launch that uses the same workspace later, unless those take more room.  sp.n_panel: the counters, sp.first_panel: the tiles.
constexpr int BLOCK_PART_BYTES = 65536, BLOCK_TILES_PER_SLOT = EPARA_BLOCK_TILES_PER_SLOT, BLOCK_COUNTER_BITS = 32 / EPARA_BLOCK_TILES_PER_COUNTER;
static_assert(BLOCK_TILES_PER_SLOT * SPLIT_MAX_PARTS * BLOCK_PART_BYTES <= SPLIT_MAX_PARTS * PANEL_SPLIT_STRIDE, "a slot is too small");
static_assert(SPLIT_MAX_PARTS < (1 << BLOCK_COUNTER_BITS), "a tile's bits of a counter hold its parts");
__device__ __forceinline__ char* block_partials(const split_ctx& sp, int tile)
{
    return panel_partials(sp) + static_cast<size_t>(tile / BLOCK_TILES_PER_SLOT) * (SPLIT_MAX_PARTS * PANEL_SPLIT_STRIDE) +
           (tile % BLOCK_TILES_PER_SLOT) * (SPLIT_MAX_PARTS * BLOCK_PART_BYTES);
}

// entry: the visit; in plain bf16 launches a tile of a long K may be visited in parts (EPARA_BLOCK_SPLIT_K).  A part leaves its raw sums in the
// workspace, lane by lane as they sit in the registers, written through to memory, and counts itself at the tile; whoever
// counts last adds the parts in index order (its own too: the order does not depend on who it is), runs the epilogue and
// puts the counter back to zero.  Nobody waits for another workgroup.
// ONCE: no other tile reads the weights (a group of a single row tile).
template <int DT, bool GATED, int FM, bool ONCE = false>
__device__ __forceinline__ void block_tile(const epara_group_args& ga, const epara_tile& tl, int entry, int out_dtype, char* lds, const split_ctx& sp)
{
    constexpr int ESZ = DT == EPARA_BF16 ? 2 : 1;
    constexpr int EPC = 16 / ESZ;                                // elements per 16-byte chunk
    constexpr int KF = 4 * EPC;                                  // K elements per stage
    constexpr int SLOT = FM * 4096;                              // bytes of a pair: FM x 32 rows x 128 bytes
    constexpr int LOADS = FM + 4;                                // a wave's loads per pair
    int tid = threadIdx.x;
    asm volatile("" : "+v"(tid));                                // what is derived from it is computed per tile
    const int lane = tid & 63;
    const int wave = __builtin_amdgcn_readfirstlane(tid >> 6);
    const int r32 = lane & 31, h = lane >> 5;
    ldsptr l3 = (ldsptr)lds;
    const int K = ga.K, N = ga.N, rows = tl.rows, cols = tl.cols;
    const int KSP = ((K + KF - 1) / KF + 3) & ~3;
    // a visit to the whole tile, or to a part of its K: whole units of two pairs.  Where the launch brought no room for the parts'
    // sums (or an entry is none of a planner's), the first visit multiplies the whole K.
    constexpr bool HAS_SPLIT = DT == EPARA_BF16 && !GATED;
    int parts = order_parts(entry), part = 0, slot_tile = 0, first_pair = 0, n_pairs = KSP >> 1;
    if (parts > 1) {
        bool room = false;
        part = order_part(entry);
        if constexpr (HAS_SPLIT) {
            const uint32_t units = static_cast<uint32_t>(KSP >> 2);
            slot_tile = ga.reserved + (tl.m0 >> 7) * ((N + 127) >> 7) + (tl.n0 >> 7);
            room = sp.ws != nullptr && parts <= SPLIT_MAX_PARTS && ga.reserved >= 0 && slot_tile < sp.first_panel && static_cast<uint32_t>(parts) <= units;
            if (room) {
                first_pair = 2 * static_cast<int>(units * part / parts);
                n_pairs = 2 * static_cast<int>(units * (part + 1) / parts) - first_pair;
            }
        }
        if (!room) parts = 1;
        if (part >= parts) return;
    }

    // ---- activations: instruction j of a pair covers rows 8 (4 j + wave) .. + 7; lane l writes chunk l % 8 of row l / 8
    // and fetches the chunk that belongs there (chunk ^ (row / 2) % 8: fragment reads are free of bank conflicts)
    const __amdgpu_buffer_rsrc_t xrsrc = __builtin_amdgcn_make_buffer_rsrc(
        const_cast<char*>(static_cast<const char*>(ga.X)) + static_cast<size_t>(tl.m0) * K * ESZ + first_pair * 128, 0, -1, 0x00020000);
    const int K_left = K - first_pair * 2 * KF;                  // of the visit; its first chunk is inside K
    const int x_chunk = (lane & 7) ^ ((4 * (wave & 1) + (lane >> 4)) & 7);
    uint32_t x_off[FM];
#pragma unroll
    for (int j = 0; j < FM; ++j)
        x_off[j] = static_cast<uint32_t>(min(8 * (4 * j + wave) + (lane >> 3), rows - 1)) * static_cast<uint32_t>(K * ESZ) + static_cast<uint32_t>(x_chunk * 16);
    // ---- weights: lane (r32, h) takes chunk 2 s2 + h of column r32 % 16 of one of the wave's two packed column blocks
    const int NB = (N + 15) >> 4, nb0 = (tl.n0 >> 4) + (GATED ? wave : 2 * wave);
    const int nb = min(GATED ? nb0 : nb0 + (r32 >> 4), NB - 1);  // a block past N only feeds columns that are not stored
    gcptr wp = as_global<char>((GATED && r32 >= 16) ? ga.W2 : ga.W) + static_cast<size_t>(nb) * KSP * 1024 +
               static_cast<size_t>(first_pair) * 2048 + (h * 16 + (r32 & 15)) * 16;

    auto w_load = [&](int i) -> v4i { return ONCE ? ld16_once(wp + i * 512) : ld16(wp + i * 512); };
    v4i w[BLOCK_RING][4];                                        // [pair % 4][2 stage + half of its K]
    auto x_issue = [&](int p, int slot, int j) {
        const int left = K_left - p * 2 * KF;                    // elements of K from this pair on
        uint32_t off = x_off[j];
        int so = p * 128;
        if (left < 2 * KF) {                                     // last pair(s) of a ragged K: chunks past K come from chunk 0
            if (x_chunk * EPC >= left) off -= static_cast<uint32_t>(x_chunk * 16);
            if (left <= 0) so = 0;
        }
        __builtin_amdgcn_raw_ptr_buffer_load_lds(xrsrc, (__attribute__((address_space(3))) void*)(l3 + slot * SLOT + (4 * j + wave) * 1024),
                                                 16, off, so, 0, 0);
    };
    auto issue = [&](int p, auto slot_tag, auto nx_tag) {        // a pair at once (the start of a tile): NX of its activation loads, its weights
        constexpr int slot = decltype(slot_tag)::value & (BLOCK_RING - 1), NX = decltype(nx_tag)::value;
#pragma unroll
        for (int j = 0; j < NX; ++j) x_issue(p, slot, j);
#pragma unroll
        for (int i = 0; i < 4; ++i) w[slot][i] = w_load(i);
        wp += 2048;
        __builtin_amdgcn_sched_barrier(0);
    };

    v16f acc[FM];
#pragma unroll
    for (int fm = 0; fm < FM; ++fm)
#pragma unroll
        for (int v = 0; v < 16; ++v) acc[fm][v] = 0.f;
    // ---- one step multiplies the K of IPS weight registers (bf16: half a stage, fp8: a stage) with the FM fragments
    // read during the step before, reads those of the next step and issues its share of the loads four pairs ahead:
    // weights into the registers just used, activations into the slot freed at the last meeting, i.e. x(p + 4, 0) at the
    // last step of pair p (fp8: 0 and 1) and the rest of them during pair p + 1.  A memory instruction or two between
    // two products, pinned by the scheduling barriers.
    constexpr int IPS = DT == EPARA_BF16 ? 1 : 2, STEPS = 4 / IPS;
    v4i xf[2][IPS][FM];
    const int sw = (r32 >> 1) & 7;
    const ldsptr xbase = l3 + r32 * 128;
    uint32_t xf_off[4];
#pragma unroll
    for (int i = 0; i < 4; ++i) xf_off[i] = static_cast<uint32_t>(((2 * i + h) ^ sw) << 4);
    auto frag = [&](int slot, int i, int fm) -> v4i { return *reinterpret_cast<lds_v4i>(xbase + slot * SLOT + xf_off[i] + fm * 4096); };
    // MODE: 0 = loads go on; the last four pairs of a tile: 1 = only the rest of the last pair's activations, 2 = none,
    // 3 = none and no next pair.  WAIT: how many loads may still be in flight when the next pair must have landed
    // (0: at least 2 FM + 8 have been issued after its last activation load; 1: 2 FM + 6; 2, first time: FM + 2).
    auto step = [&](int p, auto slot_tag, auto s_tag, auto mode_tag, auto wait_tag) {
        constexpr int slot = decltype(slot_tag)::value & (BLOCK_RING - 1), S = decltype(s_tag)::value, MODE = decltype(mode_tag)::value;
        constexpr bool LAST = S == STEPS - 1;
        constexpr int set = S & 1, nslot = LAST ? (slot + 1) & (BLOCK_RING - 1) : slot, NS = LAST ? 0 : S + 1;
        if constexpr (LAST && MODE < 3) {
            wait_lgkmcnt0();                                     // every fragment of this pair is in registers
            wait_vmcnt<decltype(wait_tag)::value>();                       // my part of the next pair has landed
            asm volatile("" ::: "memory");
            __builtin_amdgcn_s_barrier();
            asm volatile("" ::: "memory");
        }
        // activations of the pair four ahead: instruction j at the steps that follow the meeting
        constexpr int J0 = LAST ? 0 : (S + 1) * IPS;
#pragma unroll
        for (int fm = 0; fm < FM; ++fm) {
            if constexpr (DT == EPARA_BF16) mma32<DT>(acc[fm], w[slot][S], xf[set][0][fm]);
            else {
                typedef int v8i __attribute__((ext_vector_type(8)));
                acc[fm] = __builtin_amdgcn_mfma_scale_f32_32x32x64_f8f6f4(
                    __builtin_shufflevector(w[slot][S * IPS], w[slot][S * IPS + IPS - 1], 0, 1, 2, 3, 4, 5, 6, 7),
                    __builtin_shufflevector(xf[set][0][fm], xf[set][IPS - 1][fm], 0, 1, 2, 3, 4, 5, 6, 7), acc[fm], 0, 0, 0, 0, 0, 0);
            }
            if constexpr (!(LAST && MODE == 3)) {
                // two fragments after each of the first products, so that they arrive under the rest
#pragma unroll
                for (int k = 0; k < 2; ++k)
                    if (2 * fm + k < FM) {
#pragma unroll
                        for (int e = 0; e < IPS; ++e) xf[set ^ 1][e][2 * fm + k] = frag(nslot, NS * IPS + e, 2 * fm + k);
                    }
            }
            if constexpr (MODE == 0 || (MODE == 1 && !LAST)) {
                if (fm == (FM > 2 ? 2 : FM - 1)) {
#pragma unroll
                    for (int j = J0; j < J0 + IPS; ++j)
                        if (j < FM) x_issue(LAST ? p + 4 : p + 3, LAST ? slot : (slot + 3) & (BLOCK_RING - 1), j);
                }
            }
            if constexpr (MODE == 0) {
                if (fm == FM - 1) {
#pragma unroll
                    for (int e = 0; e < IPS; ++e) w[slot][S * IPS + e] = w_load(S * IPS + e);
                    if (LAST) wp += 2048;
                }
            }
            __builtin_amdgcn_sched_barrier(0);
        }
    };
    auto pair = [&](int p, auto slot_tag, auto mode_tag, auto wait_tag) {
        step(p, slot_tag, act_tag<0>{}, mode_tag, wait_tag);
        step(p, slot_tag, act_tag<1>{}, mode_tag, wait_tag);
        if constexpr (STEPS == 4) {
            step(p, slot_tag, act_tag<2>{}, mode_tag, wait_tag);
            step(p, slot_tag, act_tag<3>{}, mode_tag, wait_tag);
        }
    };
    auto first_fragments = [&](auto slot_tag) {                  // of the first pair, once it has landed for everybody
        constexpr int slot = decltype(slot_tag)::value;
        asm volatile("" ::: "memory");
        __builtin_amdgcn_s_barrier();
        asm volatile("" ::: "memory");
#pragma unroll
        for (int e = 0; e < IPS; ++e)
#pragma unroll
            for (int fm = 0; fm < FM; ++fm) xf[0][e][fm] = frag(slot, e, fm);
        __builtin_amdgcn_sched_barrier(0);
    };
    typedef act_tag<0> t0; typedef act_tag<1> t1; typedef act_tag<2> t2; typedef act_tag<3> t3;
    const act_tag<FM> all{};
    const act_tag<(FM < IPS ? FM : IPS)> head{};                 // of pair 3: the others follow during pair 0
    const act_tag<2 * LOADS> steady{};
    constexpr int AT_START = 4 + 2 * LOADS + decltype(head)::value + 4;      // loads after the first pair's activations
    if (n_pairs == 2) {                                          // K of at most 256 bytes
        issue(0, t0{}, all);
        issue(1, t1{}, all);
        wait_vmcnt<LOADS>();
        first_fragments(t0{});
        pair(0, t0{}, t2{}, act_tag<0>{});
        pair(1, t1{}, t3{}, act_tag<0>{});
    } else {
        // slots are compile-time constants, so the last four pairs sit in slots 0 .. 3: an n_pairs that is not a multiple of
        // four starts with slot 2
        int p = 0;
        if (n_pairs & 2) {
            issue(0, t2{}, all); issue(1, t3{}, all); issue(2, t0{}, all); issue(3, t1{}, head);
            wait_vmcnt<AT_START>();
            first_fragments(t2{});
            pair(0, t2{}, t0{}, steady);
            pair(1, t3{}, t0{}, steady);
            p = 2;
        } else {
            issue(0, t0{}, all); issue(1, t1{}, all); issue(2, t2{}, all); issue(3, t3{}, head);
            wait_vmcnt<AT_START>();
            first_fragments(t0{});
        }
        for (; p + 8 <= n_pairs; p += 4) {
            pair(p, t0{}, t0{}, steady);
            pair(p + 1, t1{}, t0{}, steady);
            pair(p + 2, t2{}, t0{}, steady);
            pair(p + 3, t3{}, t0{}, steady);
        }
        pair(p, t0{}, t1{}, act_tag<2 * FM + 4>{});
        pair(p + 1, t1{}, t2{}, act_tag<FM>{});
        pair(p + 2, t2{}, t2{}, act_tag<0>{});
        pair(p + 3, t3{}, t3{}, act_tag<0>{});
    }

    // ---- epilogue: act / gating in registers (a lane holds columns 8 g + 4 h .. + 3 of its wave's 32, row fm * 32 + r32),
    // then through the LDS, so that a store instruction covers whole row pieces of 256 bytes.  16-byte chunk c of a
    // row sits at c ^ (row % chunks per row).
    __syncthreads();                                             // the ring has been read
    if constexpr (HAS_SPLIT) if (parts > 1) {
        char* slab = block_partials(sp, slot_tile);
        const __amdgpu_buffer_rsrc_t rsrc = __builtin_amdgcn_make_buffer_rsrc(slab, 0, -1, 0x00020000);
        const int at = wave * 16384 + lane * 16;
#pragma unroll
        for (int fm = 0; fm < FM; ++fm)
#pragma unroll
            for (int g = 0; g < 4; ++g) {
                const v4f q = {acc[fm][4 * g], acc[fm][4 * g + 1], acc[fm][4 * g + 2], acc[fm][4 * g + 3]};
                __builtin_amdgcn_raw_buffer_store_b128(__builtin_bit_cast(v4i, q), rsrc, at, part * BLOCK_PART_BYTES + (fm * 4 + g) * 1024, 16);   // 16: device scope (sc1)
            }
        asm volatile("" ::: "memory");
        wait_vmcnt<0>();
        __syncthreads();                                         // every wave's sums are in memory
        __attribute__((address_space(3))) uint32_t* box = (__attribute__((address_space(3))) uint32_t*)l3;
        uint32_t* counter = sp.ws + sp.n_split + slot_tile / EPARA_BLOCK_TILES_PER_COUNTER;
        const int shift = slot_tile % EPARA_BLOCK_TILES_PER_COUNTER * BLOCK_COUNTER_BITS;
        if (tid == 0) *box = (__hip_atomic_fetch_add(counter, 1u << shift, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT) >> shift) & ((1u << BLOCK_COUNTER_BITS) - 1);
        __syncthreads();
        const bool last = *box == static_cast<uint32_t>(parts - 1);
        __syncthreads();                                         // the box's place in the LDS is free again
        if (!last) return;
        if (tid == 0) (void)__hip_atomic_fetch_sub(counter, static_cast<uint32_t>(parts) << shift, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT);
        auto add = [&](auto n_tag) {
            constexpr int P = decltype(n_tag)::value;
#pragma unroll
            for (int fm = 0; fm < FM; ++fm) {
                v4i in[4][P];
#pragma unroll
                for (int g = 0; g < 4; ++g)
#pragma unroll
                    for (int j = 0; j < P; ++j)
                        in[g][j] = __builtin_amdgcn_raw_buffer_load_b128(rsrc, at, j * BLOCK_PART_BYTES + (fm * 4 + g) * 1024, 16);
#pragma unroll
                for (int g = 0; g < 4; ++g) {
                    v4f sum = __builtin_bit_cast(v4f, in[g][0]);
#pragma unroll
                    for (int j = 1; j < P; ++j) sum += __builtin_bit_cast(v4f, in[g][j]);
#pragma unroll
                    for (int i = 0; i < 4; ++i) acc[fm][4 * g + i] = sum[i];
                }

            }
        };
        if (parts == 2)      add(act_tag<2>{});
        else if (parts == 3) add(act_tag<3>{});
        else                 add(act_tag<4>{});
        // nothing is in flight here; said, because a load that the compiler takes for pending on some path makes the K loop of
        // every later tile wait for all its loads once a round (2 us per launch)
        wait_vmcnt<0>();
    }
    auto finish = [&](auto out_tag, auto act) {
        constexpr int OUT = decltype(out_tag)::value, ACT = decltype(act)::value;
        constexpr int OSZ = OUT == EPARA_BF16 ? 2 : 1;
        constexpr int BN = GATED ? 64 : 128, NCH = BN * OSZ / 16;
        constexpr int WCOLS = GATED ? 16 : 32, QUADS = GATED ? 2 : 4;
        const float sg = ga.scale, s2g = ga.scale2 * ga.out_inv_scale, inv = ga.out_inv_scale;
        v4f b4[QUADS];
#pragma unroll
        for (int g = 0; g < QUADS; ++g) {
            b4[g] = v4f{0.f, 0.f, 0.f, 0.f};
            if constexpr (!GATED) {
                const int nl = wave * WCOLS + 8 * g + 4 * h;
                if (ga.bias) {
                    const EPARA_GLOBAL float* bp = as_global<float>(ga.bias) + tl.n0 + nl;
                    if (nl + 3 < cols) b4[g] = *reinterpret_cast<const EPARA_GLOBAL v4f*>(bp);
                    else {
#pragma unroll
                        for (int i = 0; i < 4; ++i) if (nl + i < cols) b4[g][i] = bp[i];
                    }
                }
            }
        }
#pragma unroll
        for (int fm = 0; fm < FM; ++fm)
#pragma unroll
            for (int g = 0; g < QUADS; ++g) {
                float v[4];
#pragma unroll
                for (int i = 0; i < 4; ++i) {
                    if constexpr (GATED) v[i] = act_fast<EPARA_ACT_SILU>(sg * acc[fm][4 * g + i]) * (s2g * acc[fm][8 + 4 * g + i]);
                    else                 v[i] = act_fast<ACT>(sg * acc[fm][4 * g + i] + b4[g][i]) * inv;
                }
                const int row = fm * 32 + r32, byte = (wave * WCOLS + 8 * g + 4 * h) * OSZ;
                ldsptr at = l3 + row * (NCH * 16) + (((byte >> 4) ^ (row & (NCH - 1))) << 4) + (byte & 15);
                if constexpr (OUT == EPARA_BF16) {
                    typedef float v2f __attribute__((ext_vector_type(2)));
                    typedef __bf16 v2bf __attribute__((ext_vector_type(2)));
                    v2u pk;
                    pk[0] = __builtin_bit_cast(uint32_t, __builtin_convertvector((v2f{v[0], v[1]}), v2bf));
                    pk[1] = __builtin_bit_cast(uint32_t, __builtin_convertvector((v2f{v[2], v[3]}), v2bf));
                    *reinterpret_cast<__attribute__((address_space(3))) v2u*>(at) = pk;
                } else {
                    *reinterpret_cast<__attribute__((address_space(3))) uint32_t*>(at) = f32x4_to_e4m3(v[0], v[1], v[2], v[3]);
                }
            }
        __syncthreads();
        constexpr int RPI = NT / NCH, EPO = 16 / OSZ;            // rows per pass over the threads, elements per chunk
        const int ch = tid % NCH, col = ch * EPO;
        const bool vec_ok = (static_cast<uint32_t>(N) * OSZ) % 16 == 0 && col + EPO <= cols;
        EPARA_GLOBAL char* y = as_global<char>(ga.Y) + (static_cast<size_t>(tl.m0) * N + tl.n0 + col) * OSZ;
#pragma unroll
        for (int r0 = 0; r0 < FM * 32; r0 += RPI) {
            const int row = r0 + tid / NCH;
            if (row >= FM * 32 || row >= rows || col >= cols) continue;
            const v4i q = *reinterpret_cast<lds_v4i>(l3 + row * (NCH * 16) + ((ch ^ (row & (NCH - 1))) << 4));
            EPARA_GLOBAL char* yr = y + static_cast<size_t>(row) * N * OSZ;
            if (vec_ok) *reinterpret_cast<EPARA_GLOBAL v4i*>(yr) = q;
            else {
#pragma unroll
                for (int e = 0; e < EPO; ++e)
                    if (col + e < cols) {
                        const uint32_t word = static_cast<uint32_t>(q[e * OSZ / 4]);
                        if constexpr (OSZ == 2) reinterpret_cast<EPARA_GLOBAL uint16_t*>(yr)[e] = static_cast<uint16_t>(word >> (16 * (e & 1)));
                        else                    reinterpret_cast<EPARA_GLOBAL uint8_t*>(yr)[e] = static_cast<uint8_t>(word >> (8 * (e & 3)));
                    }
            }
        }
    };
    auto by_out = [&](auto act) {
        if (DT == EPARA_BF16 || out_dtype == EPARA_BF16) finish(act_tag<EPARA_BF16>{}, act);
        else if constexpr (DT != EPARA_BF16)              finish(act_tag<EPARA_FP8_E4M3>{}, act);
    };
    if constexpr (GATED) by_out(act_tag<EPARA_ACT_SILU>{});
    else                 with_act(ga.act, by_out);
    __syncthreads();                                             // the next tile's activations land where the outputs were parked
}

template <int DT, bool GATED>
__global__ __launch_bounds__(NT, 2) void grouped_block_kernel(const epara_group_args* __restrict__ args, const epara_tile* __restrict__ tiles,
                                                              const int32_t* __restrict__ order, long n_slots, int out_dtype,
                                                              uint32_t* split_ws, int n_split, int n_counters, int n_tiles, int once)
{
    const split_ctx sp = {split_ws, n_split, n_counters, n_tiles};
    extern __shared__ __attribute__((aligned(16))) char lds[];
    for (long s = blockIdx.x; s < n_slots; s += gridDim.x) {
        const int t = order[s];
        if (t < 0) continue;
        const epara_tile tl = tiles[order_tile(t)];
        if (tl.cls < N_STREAM_CLASSES) continue;                 // the streaming tiles of the launch have a kernel of their own
        const epara_group_args ga = args[tl.group];
        const int fm = (tl.rows + 31) >> 5;
        if (once && ga.M <= EPARA_BLOCK_ROWS) {                  // and more than 64
            if (fm > 3)   block_tile<DT, GATED, 4, true>(ga, tl, t, out_dtype, lds, sp);
            else          block_tile<DT, GATED, 3, true>(ga, tl, t, out_dtype, lds, sp);
        }
        else if (fm > 3)  block_tile<DT, GATED, 4>(ga, tl, t, out_dtype, lds, sp);
        else if (fm == 3) block_tile<DT, GATED, 3>(ga, tl, t, out_dtype, lds, sp);
        else if (fm == 2) block_tile<DT, GATED, 2>(ga, tl, t, out_dtype, lds, sp);
        else              block_tile<DT, GATED, 1>(ga, tl, t, out_dtype, lds, sp);
    }
}

template <int DT, bool GATED>
hipError_t enqueue_block(unsigned grid, hipStream_t stream, const epara_group_args* args, const epara_tile* tiles,
                         const int32_t* order, long n_slots, int out_dtype, uint32_t* split_ws, int n_split, int n_counters, int n_tiles, int once)
{
    static const hipError_t attr = hipFuncSetAttribute(reinterpret_cast<const void*>(&grouped_block_kernel<DT, GATED>),
                                                       hipFuncAttributeMaxDynamicSharedMemorySize, BLOCK_LDS_BYTES);
    if (attr != hipSuccess) return attr;
    hipLaunchKernelGGL((grouped_block_kernel<DT, GATED>), dim3(grid), dim3(NT), BLOCK_LDS_BYTES, stream, args, tiles, order, n_slots, out_dtype, split_ws, n_split, n_counters, n_tiles, once);
    return hipGetLastError();
}

}  // namespace

#endif
