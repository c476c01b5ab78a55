// decode_byzantine_pairs_kernel with Algorithm 1's locator, K + A = 13 and 14; a source file of its own for the build's sake.
#include "byzantine_pairs.h"

namespace approxifer {
int run_null_pairs_14(int tq, const PairCall &call, const Nodes &nodes, hipStream_t stream) {
    return run_pairs_columns<14, true>(tq, call, nodes, stream);
}
}  // namespace approxifer
