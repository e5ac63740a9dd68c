// C interface to the admission arithmetic of the serving loop.
#include "serve_core.h"

extern "C" {
int64_t at_once(int64_t m, int64_t chunk, int32_t streams) { return stag::serve::chunks_at_once(m, chunk, streams); }
uint64_t allowance(uint64_t budget, int32_t streams, int64_t chunk, int64_t m, uint64_t base, uint64_t need) {
  return stag::serve::chunk_allowance(budget, streams, chunk, m, base, need);
}
}
