// The R W products of passes_full.h, and the choice between them and the products of passes.hip.
#include "passes_full.h"

#define FULL_LONG 8192
int full_blocks(int n, int LP) { return ceil_div(n, 16 * full_group(n, LP)); }
int full_blocks_most(int n, int LP) { return max(min(256, ceil_div(n, 16)), full_blocks(min(n, FULL_LONG), LP)); }

// Ranges of the reduction; 0: the products of passes.hip.  It depends on the operand's own sizes alone (a factor's bits do not
// depend on the other operand), so that an operand takes the same form beside any other; and all operands of the calls below 13
// million elements are taken, so that no step of theirs needs two launches: one operand in each form cost 500 x 500 x 1800, 24
// columns 166 us in place of 150.
// One power iteration, us per call, passes.hip / here, by sketch columns:
//   200^3                 10 66.5 / 54.1   24 126 / 108   40 179 / 158
//   1000^3                10 85 / 75.5     24 148 / 131   40 205 / 186   80 387 / 370
//   2000^3                10 130 / 113     24 201 / 166   40 267 / 230   80 465 / 426
//   2700^3                                 24 247 / 219   40 322 / 297   80 549 / 530
//   256 x 512 x 8192      8 144 / 141      24 199 / 195   40 285 / 271   80 517 / 501
//   128 x 128 x 4096      8 100 / 89       24 150 / 149   40 224 / 211   80 426 / 415
// Calls with two chains, the large operand's form / here too: 4096^3 24 330 / 329, 40 398 / 398, 80 635 / 694, 1024 x 4096 x 4096 24
// 254 / 262, 40 324 / 334: operands above 16.2 million elements stay there, but for one tile of sketch columns (10 275 / 270).
// Small operands beside one of those, all passes.hip / here: 1024 x 4096 x 4096 24 254 / 254, 40 325 / 324, 80 556 / 565; 4096 x 512 x
// 4096 24 224 / 231, 40 291 / 293; 3900 x 300 x 4096 24 224 / 225, 40 295 / 296: the one at 24 columns is slower.
// Operands with a side beyond 8192 stay there (500 x 300 x 12000 l = 24 252 / 275; a step of such a call would take two
// launches), but for the transposed product of a tall one (100352 x 64 x 64 l = 8 111 / 99).
// Long reductions are cut, into ranges of 512 and more as long as there are CUs without a workgroup, whole / cut: 300 x 5000 x
// 1200 l = 8 113 / 110, 40 236 / 226; 6000 x 300 x 300 l = 8 104 / 82; not below 84 steps: 2000^3 l = 24 173 whole, 183 cut in
// two.  FULL_BLOCKS is a constant, and not the device's count of CUs, since the ranges decide the order of addition.
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
