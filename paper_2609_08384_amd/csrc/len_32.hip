// Pass launchers of plans, batches and the adjoint for the line lengths 8x4
// (N1 x N2; see launch.hpp and lengths.hpp).
#include "launch_impl.hpp"

BRAHMS_INSTANTIATE_LENGTH(8, 4)
