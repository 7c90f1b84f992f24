// Pass launchers of plans and batches for the second splits 8x1 12x1
// (N1 x N2; see launch.hpp and lengths.hpp).
#include "launch_impl.hpp"

BRAHMS_INSTANTIATE_PASSES(8, 1)
BRAHMS_INSTANTIATE_PASSES(12, 1)
