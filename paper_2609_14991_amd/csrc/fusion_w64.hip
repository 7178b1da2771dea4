#include "fusion_device.h"

namespace fusion {
KernelFn pick_w64(int km, bool al, int mode) { return pick_k<64, 1, 1>(km, al, mode); }
}  // namespace fusion
