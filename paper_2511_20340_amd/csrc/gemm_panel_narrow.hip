// The panel kernel's smaller tiles (the list: gemm_panel.hip).
#include "gemm_panel.h"

namespace sf {

hipError_t dispatch_panel_narrow(int tile, const GemmArgs &a, hipStream_t s, int split) {
  switch (tile) {
    case 18: return run_panel<2, 2, 4, 8, 3>(a, s, split);
    case 26: return run_panel<2, 2, 4, 4, 4>(a, s, split);
    case 27: return run_panel<2, 2, 5, 4, 2>(a, s, split);
    case 28: return run_panel<2, 2, 5, 4, 4>(a, s, split);
    default: return hipErrorInvalidValue;
  }
}

hipError_t prepare_panel_narrow() {
  hipError_t err = ensure_panel_lds<2, 2, 4, 8, 3>();
  if (err == hipSuccess) err = ensure_panel_lds<2, 2, 5, 4, 4>();
  if (err == hipSuccess) err = ensure_panel_lds<2, 2, 4, 4, 4>();
  if (err == hipSuccess) err = ensure_panel_lds<2, 2, 5, 4, 2>();
  return err;
}

}  // namespace sf
