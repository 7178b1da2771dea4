#include "fusion_device.h"

namespace fusion {
KernelFn pick_w64_2lm(int km, bool al, int mode) { return pick_k<64, 1, 2>(km, al, mode); }
}  // namespace fusion
