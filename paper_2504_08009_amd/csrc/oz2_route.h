// Rules of the launches that oz2_host_route tells too.
#ifndef OZ2_ROUTE_H
#define OZ2_ROUTE_H

#include "oz2_internal.h"

// The operand (1, 2; 0: neither) that the one-pass conversion takes alone, beside separate launches for the other, where
// oz2_one_pass_vectors says 0.  lines_a, lines_b: as it takes them; triangular: one of the operands is.
int oz2_one_pass_operand(const Oz2Plan& plan, const Oz2Layout& lay, int strided_a, int strided_b, int lines_a, int lines_b, int triangular,
                         int symmetric, int shift_mode, int bit_split, int64_t cus);
// Are the residue planes of a one-pass conversion of both operands stored through the caches?
bool oz2_planes_through_caches(int num_moduli, const Oz2Layout& lay, int64_t m, int64_t n, bool symmetric);
// Is line 9 formed on the matrix cores?  triangle: 0, 1 or 2, as oz2_launch_stage3 takes it.
bool oz2_crt_on_matrix_cores(const Oz2Plan& plan, int64_t m, int64_t n, int residue_u8, int triangle);

#endif
