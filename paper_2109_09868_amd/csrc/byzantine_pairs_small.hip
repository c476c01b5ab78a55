// decode_byzantine_pairs_kernel for up to eight columns (K + A <= 8); a source file of its own for the build's sake.
#include "byzantine_pairs.h"

namespace approxifer {
int run_pairs_4(int missing, int extra, const PairCall &call, int nw, const Nodes &nodes, hipStream_t stream) {
    return run_pairs_columns<4>(missing, extra, call, nw, nodes, stream);
}
int run_pairs_6(int missing, int extra, const PairCall &call, int nw, const Nodes &nodes, hipStream_t stream) {
    return run_pairs_columns<6>(missing, extra, call, nw, nodes, stream);
}
int run_pairs_8(int missing, int extra, const PairCall &call, int nw, const Nodes &nodes, hipStream_t stream) {
    return run_pairs_columns<8>(missing, extra, call, nw, nodes, stream);
}
}  // namespace approxifer
