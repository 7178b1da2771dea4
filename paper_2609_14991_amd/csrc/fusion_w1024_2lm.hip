#include "fusion_device.h"

namespace fusion {
KernelFn pick_w1024_2lm(int km, bool al, int mode) { return pick_k<1024, 1, 2>(km, al, mode); }
}  // namespace fusion
