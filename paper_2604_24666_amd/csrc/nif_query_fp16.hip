// The fused query with FP16 MLP arithmetic.
#include "nif_query.hpp"

namespace nif {

int query_fp16(const QueryShape& sh, int hw, const NetParams& np, const GridArgs& G, const RayArgs& R, const nif_hits& out,
               int64_t* ctr, int64_t* stats, int pt, hipStream_t st) {
    return dispatch_query<P_FP16>(sh, hw, np, G, R, out, ctr, stats, pt, st);
}

}  // namespace nif
