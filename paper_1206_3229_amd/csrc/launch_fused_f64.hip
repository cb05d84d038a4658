// Kernel launchers of the library, one translation unit per kernel family
// (compiled in parallel); declared in vlasov_internal.hpp.
#include "launch_fused.hpp"

namespace vlasov_detail {

template int launch_kick_drift<double>(vlasov_ctx *, int, bool, int64_t, double);

}  // namespace vlasov_detail
