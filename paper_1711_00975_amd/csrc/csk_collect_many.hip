// csk_collect_many.hip — the collect kernel (csk_collect_body.h) for sketches of 6 to 8 rows.
#include <hip/hip_runtime.h>
#include <stdint.h>

#include "csk_collect_body.h"

namespace csk {

using namespace collect2;

void launch_collect2_many(uint32_t d, uint32_t mode, int hm, dim3 grid, dim3 block, size_t lds, hipStream_t s,
                          const CollectLaunch& c) {
  switch (d) {
    case 6: launch_collect2_dm<6>(mode, hm, grid, block, lds, s, c); break;
    case 7: launch_collect2_dm<7>(mode, hm, grid, block, lds, s, c); break;
    default: launch_collect2_dm<8>(mode, hm, grid, block, lds, s, c); break;
  }
}

}  // namespace csk
