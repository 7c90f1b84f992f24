// Pass launchers of plans, batches and the adjoint for the line lengths 1x1 2x1 3x1 4x1 6x1
// (N1 x N2; see launch.hpp and lengths.hpp).
#include "launch_impl.hpp"

BRAHMS_INSTANTIATE_LENGTH(1, 1)
BRAHMS_INSTANTIATE_LENGTH(2, 1)
BRAHMS_INSTANTIATE_LENGTH(3, 1)
BRAHMS_INSTANTIATE_LENGTH(4, 1)
BRAHMS_INSTANTIATE_LENGTH(6, 1)
