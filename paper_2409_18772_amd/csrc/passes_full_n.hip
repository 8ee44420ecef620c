// The R W products of passes_full.h, and the choice between them and the products of passes.hip.
#include "passes_full.h"

#define FULL_LONG 8192
int full_blocks(int n, int LP) { return ceil_div(n, 16 * full_group(n, LP)); }
int full_blocks_most(int n, int LP) { return max(min(256, ceil_div(n, 16)), full_blocks(min(n, FULL_LONG), LP)); }

// Ranges of the reduction; 0: the products of passes.hip.  It depends on the operand's own sizes alone (a factor's bits do not depend
// on the other operand), and all operands of calls that advance both factorizations together (two_chains) are taken, so that no step
// of theirs needs two launches: one operand in each form cost 500 x 500 x 1800, 24 columns 166 us in place of 150.
// One power iteration, us per call, passes.hip / here: 200^3 l = 10 66.5 / 54.1, 24 126 / 110; 1000^3 10 85 / 75.5, 24 146 / 134, 80 387 /
// 370; 2000^3 10 130 / 113, 24 198 / 173, 40 266 / 240, 80 463 / 432; two chains: 2800^3 24 242 / 232, 40 319 / 307; 3300^3 10 239 / 220, 24
// 289 / 278, 40 357 / 357; 4096^3 10 275 / 270, 24 319 / 345, 40 393 / 450, 80 629 / 689: workgroups that take a CU for themselves keep the other
// chain's kernels out.  So the operands of calls with two chains stay, but for one tile of sketch columns; see two_chains for where
// both advance together, which is better than either.
// Operands with a side beyond 8192 stay there (500 x 300 x 12000 l = 24 252 / 275; a step of such a call would take two launches), but for the
// transposed product of a tall one (100352 x 64 x 64 l = 8 111 / 99).
// Long reductions are cut, into ranges of 512 and more as long as there are CUs without a workgroup, whole / cut: 300 x 5000 x 1200 l = 8
// 113 / 110, 40 236 / 226; 6000 x 300 x 300 l = 8 104 / 82; not below 84 steps: 2000^3 l = 24 173 whole, 183 cut in two.
#define FULL_CUT 84
#define FULL_BLOCKS 256
int pass_full_ranges(bool t_type, int rows, int cols, int ldx, int LP) {
    const int n = t_type ? cols : rows, len = t_type ? rows : cols;
    if (ldx > (1 << 22) || len < 64 || n < 64) return 0;        // (offsets of a workgroup's rows in 32 bits)
    if (cols > FULL_LONG || (rows > FULL_LONG && !(t_type && LP == 16))) return 0;
    if ((long long)n * len > (max(n, len) <= 4096 ? FULL_ELEMENTS : 13000000)) return LP == 16 && len <= 4096;
    const int tiles = ceil_div(n, 16), steps = len >> 5;
    if (steps < FULL_CUT) return 1;
    const int most = min(max(1, min(FULL_BLOCKS / tiles, steps / 16)), MAX_SPLITS_T);
    return ceil_div(steps, ceil_div(steps, most));
}

// Up to FULL_LONG of either side, and the rows of a tall operand of up to 13 million elements with 64 columns and more beside
// sketches of 16.
size_t full_steps_bytes(int rows, int cols, int LP) {
    return max(steps_bytes(min(max(rows, cols), FULL_LONG), LP), steps_bytes(min(rows, 13000000 / 64), 16));
}

int launch_pass_full_n(const PassOperand* op, int nop, QuantParams q, int LP, hipStream_t st, int planes) {
    return launch_full_t<false>(op, nop, q, LP, st, planes);
}
