// decode_byzantine_pairs_kernel with Algorithm 2's locator, K + A up to 8; a source file of its own for the build's sake.
#include "byzantine_pairs.h"

namespace approxifer {
int run_pairs_4(int tq, const PairCall &call, const Nodes &nodes, hipStream_t stream) {
    return run_pairs_columns<4, false>(tq, call, nodes, stream);
}
int run_pairs_6(int tq, const PairCall &call, const Nodes &nodes, hipStream_t stream) {
    return run_pairs_columns<6, false>(tq, call, nodes, stream);
}
int run_pairs_8(int tq, const PairCall &call, const Nodes &nodes, hipStream_t stream) {
    return run_pairs_columns<8, false>(tq, call, nodes, stream);
}
}  // namespace approxifer
