// decode_byzantine_pairs_kernel with Algorithm 2's locator, K + A up to 12, from 9; a source file of its own for the build's sake.
#include "byzantine_pairs.h"

namespace approxifer {
int run_pairs_10(int tq, const PairCall &call, const Nodes &nodes, hipStream_t stream) {
    return run_pairs_columns<10, false>(tq, call, nodes, stream);
}
int run_pairs_12(int tq, const PairCall &call, const Nodes &nodes, hipStream_t stream) {
    return run_pairs_columns<12, false>(tq, call, nodes, stream);
}
}  // namespace approxifer
