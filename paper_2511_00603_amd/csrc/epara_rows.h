// The order in which the chunks of a batch are quantised (no HIP types: it also builds alone).
//
// Backwards in eights: up to 32 MB that the maxima kernel has read last may still be in the L2 of the die that read them, and
// workgroups go to the eight dies in turn, so chunk c runs on a workgroup that is c modulo 8, as it did there.  For that
// the grid covers whole eights: with n_chunks workgroups instead, the up to seven indices past them would wrap to workgroups of
// other residues, which take a second round for them while as many workgroups have nothing to do.
#ifndef EPARA_ROWS_H
#define EPARA_ROWS_H

#include <stdint.h>

constexpr int64_t ROWS_MAX_GRID = 256 * 16;

// How many indices the workgroups go through, index i on workgroup i modulo the grid.
constexpr int64_t quantize_span(int64_t n_chunks) { return (n_chunks + 7) & ~static_cast<int64_t>(7); }
// The chunk of index i; n_chunks or more: none.
constexpr int64_t quantize_chunk(int64_t i, int64_t n_chunks) { return quantize_span(n_chunks) - 8 - (i & ~static_cast<int64_t>(7)) + (i & 7); }
// Workgroups (one, which writes the scales, without chunks).
constexpr int64_t quantize_grid(int64_t n_chunks)
{
    return n_chunks <= 0 ? 1 : quantize_span(n_chunks) < ROWS_MAX_GRID ? quantize_span(n_chunks) : ROWS_MAX_GRID;
}

#endif
