// Kernel launchers of the library, one translation unit per kernel family
// (compiled in parallel); declared in vlasov_internal.hpp.
#include "launch_fused.hpp"

namespace vlasov_detail {

template int launch_kick_drift_w<double, 230>(vlasov_ctx *, int, double);
template int launch_kick_drift_w<double, 486>(vlasov_ctx *, int, double);

}  // namespace vlasov_detail
