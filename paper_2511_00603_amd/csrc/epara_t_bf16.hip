// Grouped launches of libepara planned with the block table: bf16 kernels.
#include "epara_block_tile.h"
#include "epara_internal.h"

hipError_t epara_enqueue_block_bf16(int gated, unsigned grid, hipStream_t stream, const epara_group_args* args, const epara_tile* tiles,
                                    const int32_t* order, long n_slots, int out_dtype, uint32_t* split_ws, int n_split, int n_counters, int n_tiles, int once)
{
    return (gated ? enqueue_block<EPARA_BF16, true> : enqueue_block<EPARA_BF16, false>)(grid, stream, args, tiles, order, n_slots, out_dtype, split_ws, n_split, n_counters, n_tiles, once);
}
