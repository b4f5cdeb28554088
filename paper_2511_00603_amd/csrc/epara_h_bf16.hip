// Grouped launches of libepara whose panel tiles are multiplied in halves: bf16 kernels.
#include "epara_half.h"
#include "epara_internal.h"

hipError_t epara_enqueue_half_bf16(int gated, unsigned n_lists, hipStream_t stream, const epara_group_args* args, const epara_tile* tiles,
                                   const int32_t* order, long n_slots, int out_dtype)
{
    return (gated ? enqueue_half<EPARA_BF16, true> : enqueue_half<EPARA_BF16, false>)(n_lists, stream, args, tiles, order, n_slots, out_dtype);
}
