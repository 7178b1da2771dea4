#include "fusion_device.h"

namespace fusion {
KernelFn pick_w1024x2(int km, bool al, int mode) { return pick_k<1024, 2, 1>(km, al, mode); }
}  // namespace fusion
