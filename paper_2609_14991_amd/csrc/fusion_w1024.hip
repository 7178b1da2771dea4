#include "fusion_device.h"

namespace fusion {
KernelFn pick_w1024(int km, bool al, int mode) { return pick_k<1024, 1, 1>(km, al, mode); }
}  // namespace fusion
