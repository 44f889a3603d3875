// csk_append_few.hip — launches of the append bin kernel (csk_append_body.h) for sketches of
// d = 1..4 rows (row-interleaved tables, any width).
#include <hip/hip_runtime.h>
#include <stdint.h>

#include "csk_append_body.h"

namespace csk {

using namespace append;

hipError_t launch_append_few(const BinArgs& a, uint32_t mode, hipStream_t s) {
  switch (a.d) {
    case 1: launch_append_d<1, true>(a, mode, s); break;
    case 2: launch_append_d<2, true>(a, mode, s); break;
    case 3: launch_append_d<3, true>(a, mode, s); break;
    default: launch_append_d<4, true>(a, mode, s); break;
  }
  return hipGetLastError();
}

hipError_t launch_append_few_batch(const AppendBatch& b, uint32_t d, uint32_t mode, uint32_t kb, hipStream_t s) {
  switch (d) {
    case 1: launch_append_batch_d<1, true>(b, mode, kb, s); break;
    case 2: launch_append_batch_d<2, true>(b, mode, kb, s); break;
    case 3: launch_append_batch_d<3, true>(b, mode, kb, s); break;
    default: launch_append_batch_d<4, true>(b, mode, kb, s); break;
  }
  return hipGetLastError();
}

}  // namespace csk
