// What the host half of libepara shares with the launch code beyond the C ABI (no HIP types: it also builds alone).
#ifndef EPARA_PLAN_H
#define EPARA_PLAN_H

#include <stdint.h>

#include "epara.h"

#define EPARA_HIDDEN __attribute__((visibility("hidden")))

// Slots (three tiles each) of the block tiles of a launch that may be visited in parts of K ("Block tiles" in the header); how
// many parts, or whether at all, is a search that only the planner makes.  Shapes and classes are valid.
EPARA_HIDDEN int32_t epara_block_slots(const epara_group_desc* groups, int32_t G, const epara_tile_class* classes, int32_t n_classes, int32_t n_stream_classes);

#endif
