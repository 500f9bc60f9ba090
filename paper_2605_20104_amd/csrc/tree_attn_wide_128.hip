// tree_attn_wide_128_kernel: the kernel of tree_attn_wide.hip on tiles of 128 rows, two wavefronts sharing 64 of them (which shapes
// take it: make_plan in tree_attn.hip).
#define GRAFT_WIDE_128
#include "tree_attn_wide.hip"
