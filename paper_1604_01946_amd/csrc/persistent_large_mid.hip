// The one-layer kernels of persistent_large_dev.h for hidden sizes between 512, 1024 and 2048 (large_mid_size).
#include "persistent_large_dev.h"

namespace lstm {

hipError_t launch_fwdL_mid(int H, int cell, const PersFwdLArgs& k, hipStream_t s, bool s3) {
  switch (H) {
    case 640: return launch_fwdL_cell<640>(cell, k, s, s3);
    case 768: return launch_fwdL_cell<768>(cell, k, s, s3);
    case 896: return launch_fwdL_cell<896>(cell, k, s, s3);
    case 1536: return launch_fwdL_cell<1536>(cell, k, s, s3);
    case 1792: return launch_fwdL_cell<1792>(cell, k, s, s3);
  }
  return hipErrorInvalidValue;
}

hipError_t launch_bwdL_mid(int H, int cell, const PersBwdLArgs& k, hipStream_t s, bool s3) {
  switch (H) {
    case 640: return k.ks == 4 ? launch_bwdL_cell<640, 4>(cell, k, s, s3) : launch_bwdL_cell<640, 2>(cell, k, s, s3);
    case 768: return k.ks == 4 ? launch_bwdL_cell<768, 4>(cell, k, s, s3) : launch_bwdL_cell<768, 2>(cell, k, s, s3);
    case 896: return k.ks == 4 ? launch_bwdL_cell<896, 4>(cell, k, s, s3) : launch_bwdL_cell<896, 2>(cell, k, s, s3);
    case 1536: return launch_bwdL_cell<1536, 1>(cell, k, s, s3);
    case 1792: return launch_bwdL_cell<1792, 1>(cell, k, s, s3);
  }
  return hipErrorInvalidValue;
}

}  // namespace lstm
