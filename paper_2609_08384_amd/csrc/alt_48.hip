// Pass launchers of plans and batches for the second splits 24x2
// (N1 x N2; see launch.hpp and lengths.hpp).
#include "launch_impl.hpp"

BRAHMS_INSTANTIATE_PASSES(24, 2)
