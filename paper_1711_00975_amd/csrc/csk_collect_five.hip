// csk_collect_five.hip — the collect kernel (csk_collect_body.h) for sketches of 5 rows.
#include <hip/hip_runtime.h>
#include <stdint.h>

#include "csk_collect_body.h"

namespace csk {

using namespace collect2;

void launch_collect2_five(uint32_t mode, int hm, dim3 grid, dim3 block, size_t lds, hipStream_t s, const CollectLaunch& c) {
  launch_collect2_dm<5>(mode, hm, grid, block, lds, s, c);
}

}  // namespace csk
