// The kernel instances of the calls whose radix passes have no count launch,
// and of small calls' mean (at most kSmallChunks filter chunks), in a code
// object of their own: with them inside the objects of the other kernels,
// five frames of 1.3 million points took 86.1 us a call instead of 85.5, every
// kernel's code the same (what is fetched for each of a call's kernels lies
// further apart).
#define MMBEV_SMALL_CALLS
#include "filter.hip"
#include "sort.hip"
#include "voxel.hip"
