// csk_collect_few.hip — the collect kernel (csk_collect_body.h) for sketches of 1 to 4 rows.
#include <hip/hip_runtime.h>
#include <stdint.h>

#include "csk_collect_body.h"

namespace csk {

using namespace collect2;

void launch_collect2_few(uint32_t d, uint32_t mode, int hm, dim3 grid, dim3 block, size_t lds, hipStream_t s,
                         const CollectLaunch& c) {
  switch (d) {
    case 1: launch_collect2_dm<1>(mode, hm, grid, block, lds, s, c); break;
    case 2: launch_collect2_dm<2>(mode, hm, grid, block, lds, s, c); break;
    case 3: launch_collect2_dm<3>(mode, hm, grid, block, lds, s, c); break;
    default: launch_collect2_dm<4>(mode, hm, grid, block, lds, s, c); break;
  }
}

}  // namespace csk
