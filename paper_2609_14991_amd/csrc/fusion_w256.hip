#include "fusion_device.h"

namespace fusion {
KernelFn pick_w256(int km, bool al, int mode) { return pick_k<256, 1, 1>(km, al, mode); }
}  // namespace fusion
