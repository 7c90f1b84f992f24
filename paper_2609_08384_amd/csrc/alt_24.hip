// Pass launchers of plans, batches and the adjoint for the second splits 24x1
// (N1 x N2; see launch.hpp and lengths.hpp).
#include "launch_impl.hpp"

BRAHMS_INSTANTIATE_LENGTH(24, 1)
