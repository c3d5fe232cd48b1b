// Kernel instances: fp32 MTTKRP.
#include "kernel_impl.h"

namespace amped {
namespace dev {

KernelFn pick_mttkrp_f32(int nin, Lanes v, bool buf) { return pick_any<float, 0>(nin, v, buf); }

}  // namespace dev
}  // namespace amped
