// The count by which a launch's last workgroup knows itself.  Plain arithmetic: no GPU is needed to check it.
#pragma once
#include <stdint.h>

// What workgroup `block` of `grid` adds to the word: 1, but the first one takes away what the others add.  The word is then 0 again when all have
// been here and, as long as it began at 0, not before; no workgroup resets it, so launches that overlap (their results are undefined) leave 0 too.  (Reset by the
// last workgroup, it lost what another launch had added in the meantime, for good.)
__host__ __device__ inline uint32_t usl_count_share(uint32_t block, uint32_t grid) { return block ? 1u : 1u - grid; }
// before: the word as the addition found it
__host__ __device__ inline bool usl_count_is_last(uint32_t before, uint32_t share) { return before + share == 0u; }
