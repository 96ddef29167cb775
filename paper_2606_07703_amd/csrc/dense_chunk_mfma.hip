// Dense causal GQA attention (dense_tile.hpp) of the query rows of a chunk.
// Built without the assumption that no value is NaN: rows that come out NaN
// are computed again.
#include "dense_tile.hpp"

namespace sp {

hipError_t launch_dense_chunk_mfma(const Prob &p, const void *q, const void *k, const void *v,
                                   void *o, float *lse, hipStream_t st) {
  return launch_dense_d<true, true>(p, q, k, v, o, lse, st);
}

}  // namespace sp
