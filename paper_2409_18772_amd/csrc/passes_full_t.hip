// The R^T Y products of passes_full.h.
#include "passes_full.h"

int launch_pass_full_t(const PassOperand* op, int nop, QuantParams q, int LP, hipStream_t st, int planes) {
    return launch_full_t<true>(op, nop, q, LP, st, planes);
}
