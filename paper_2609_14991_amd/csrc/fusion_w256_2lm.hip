#include "fusion_device.h"

namespace fusion {
KernelFn pick_w256_2lm(int km, bool al, int mode) { return pick_k<256, 1, 2>(km, al, mode); }
}  // namespace fusion
