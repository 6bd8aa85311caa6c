// Kernel instance: gg2_f64 (final gluons 2, channel 0, amplitudes in double).
// VEGAS iterations of this instance use the staged path (see mf_api.hip), and
// its integrand four lanes per event: the amplitudes of the 24 orderings of
// one event do not fit one lane's registers in FP64.
#include "kernels.h"
namespace mf {
Launchers launchers_gg2_f64() { return make_launchers<2, 0, double, Dual<double>, 0, 0, 4>(); }
}  // namespace mf
