// Kernel instances: sparse CP loss.
#include "kernel_impl.h"

namespace amped {
namespace dev {

KernelFn pick_loss(int nin, Lanes v, bool buf) { return pick_any<float, 2>(nin, v, buf); }

}  // namespace dev
}  // namespace amped
