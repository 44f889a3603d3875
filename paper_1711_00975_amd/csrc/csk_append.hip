// csk_append.hip — launches of the append bin kernel (csk_append_body.h) on the packed
// sort-word table: d = 5..8 rows and w = 2^lw counters per row with lw + 1 <= floor(128 / d).
#include <hip/hip_runtime.h>
#include <stdint.h>

#include "csk_append_body.h"

namespace csk {

using namespace append;

uint32_t append_lds_bytes(uint32_t d, uint32_t kb, uint32_t P, uint32_t ring, bool rows, bool ex) {
  const uint32_t dp = rows ? (d <= 4 ? 4u : (d <= 6 ? 6u : 8u)) : 4u;
  return append_lds(dp, kb, P, ring, ex).bytes;
}

hipError_t launch_append(const BinArgs& a, uint32_t mode, hipStream_t s) {
  if (a.plan.sort == kAppendRows) return a.d <= 4 ? launch_append_few(a, mode, s) : launch_append_rows(a, mode, s);
  switch (a.d) {
    case 5: launch_append_d<5, false>(a, mode, s); break;
    case 6: launch_append_d<6, false>(a, mode, s); break;
    case 7: launch_append_d<7, false>(a, mode, s); break;
    default: launch_append_d<8, false>(a, mode, s); break;
  }
  return hipGetLastError();
}

hipError_t launch_append_batch(const AppendBatch& b, uint32_t d, uint32_t mode, const BinPlan& form, hipStream_t s) {
  const uint32_t kb = form.kb;
  if (form.sort == kAppendRows)
    return d <= 4 ? launch_append_few_batch(b, d, mode, kb, s) : launch_append_rows_batch(b, d, mode, kb, s);
  switch (d) {
    case 5: launch_append_batch_d<5, false>(b, mode, kb, s); break;
    case 6: launch_append_batch_d<6, false>(b, mode, kb, s); break;
    case 7: launch_append_batch_d<7, false>(b, mode, kb, s); break;
    default: launch_append_batch_d<8, false>(b, mode, kb, s); break;
  }
  return hipGetLastError();
}

}  // namespace csk
