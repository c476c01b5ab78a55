// decode_byzantine_pairs_kernel for nine to fourteen columns (K + A); a source file of its own for the build's sake.
#include "byzantine_pairs.h"

namespace approxifer {
int run_pairs_10(int missing, int extra, const PairCall &call, int nw, const Nodes &nodes, hipStream_t stream) {
    return run_pairs_columns<10>(missing, extra, call, nw, nodes, stream);
}
int run_pairs_12(int missing, int extra, const PairCall &call, int nw, const Nodes &nodes, hipStream_t stream) {
    return run_pairs_columns<12>(missing, extra, call, nw, nodes, stream);
}
int run_pairs_14(int missing, int extra, const PairCall &call, int nw, const Nodes &nodes, hipStream_t stream) {
    return run_pairs_columns<14>(missing, extra, call, nw, nodes, stream);
}
}  // namespace approxifer
