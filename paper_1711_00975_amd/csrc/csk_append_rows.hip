// csk_append_rows.hip — launches of the append bin kernel (csk_append_body.h) on the
// row-interleaved tables with multiply-high buckets: d = 5..8 rows of any width, and, for
// d = 5, the update of the learned router's rest sketch with its exclusion.
#include <hip/hip_runtime.h>
#include <stdint.h>

#include "csk_append_body.h"

namespace csk {

using namespace append;

hipError_t launch_append_rows(const BinArgs& a, uint32_t mode, hipStream_t s) {
  switch (a.d) {
    case 5: launch_append_d<5, true>(a, mode, s); break;
    case 6: launch_append_d<6, true>(a, mode, s); break;
    case 7: launch_append_d<7, true>(a, mode, s); break;
    default: launch_append_d<8, true>(a, mode, s); break;
  }
  return hipGetLastError();
}

hipError_t launch_append_routed(const BinArgs& a, uint32_t mode, hipStream_t s) {
  if (mode == kMeshPow2Ratio) launch_append_kb<5, kMeshPow2Ratio, true, true>(a, s);
  else if (mode == kMeshExactRatio) launch_append_kb<5, kMeshExactRatio, true, true>(a, s);
  else launch_append_kb<5, kMeshGeneral, true, true>(a, s);
  return hipGetLastError();
}

hipError_t launch_append_rows_batch(const AppendBatch& b, uint32_t d, uint32_t mode, uint32_t kb, hipStream_t s) {
  switch (d) {
    case 5: launch_append_batch_d<5, true>(b, mode, kb, s); break;
    case 6: launch_append_batch_d<6, true>(b, mode, kb, s); break;
    case 7: launch_append_batch_d<7, true>(b, mode, kb, s); break;
    default: launch_append_batch_d<8, true>(b, mode, kb, s); break;
  }
  return hipGetLastError();
}

}  // namespace csk
