// The grouped GEMM kernel's 128-row tile, in a file of its own so that the two
// tiles compile side by side.
#include "gemm_kernel.h"

namespace moe {
namespace gemm {
namespace {
template <int MODE>
void launch(unsigned grid, const GemmArgs& a, hipStream_t s) {
  grouped_gemm_kernel<MODE, TILE_S><<<grid, Geom<TILE_S>::NTHR, 0, s>>>(a);
}
}  // namespace

void launch_small(int mode, unsigned grid, const GemmArgs& a, hipStream_t s) {
  switch (mode) {
    case FWD_GATE_UP: return launch<FWD_GATE_UP>(grid, a, s);
    case FWD_DOWN: return launch<FWD_DOWN>(grid, a, s);
    case DGRAD_DOWN: return launch<DGRAD_DOWN>(grid, a, s);
    case DGRAD_GATE_UP: return launch<DGRAD_GATE_UP>(grid, a, s);
    case WGRAD_GATE_UP: return launch<WGRAD_GATE_UP>(grid, a, s);
    case WGRAD_DOWN: return launch<WGRAD_DOWN>(grid, a, s);
    case RT_DW: return launch<RT_DW>(grid, a, s);
    case RT_DX: return launch<RT_DX>(grid, a, s);
    case VOC_FWD: return launch<VOC_FWD>(grid, a, s);
    case VOC_GRAD: return launch<VOC_GRAD>(grid, a, s);
    case VOC_DX: return launch<VOC_DX>(grid, a, s);
    case VOC_DW: return launch<VOC_DW>(grid, a, s);
  }
}

}  // namespace gemm
}  // namespace moe
