// Kernel instances: fused residual + MTTKRP gradient.
#include "kernel_impl.h"

namespace amped {
namespace dev {

KernelFn pick_grad(int nin, Lanes v, bool buf) { return pick_any<float, 1>(nin, v, buf); }

}  // namespace dev
}  // namespace amped
