// Launchers of the pass kernels, one set per line-transform length (declared
// here, defined in launch_impl.hpp, instantiated per length in len_*.hip so
// that the lengths compile in parallel).
#pragma once

#include <hip/hip_runtime.h>

#include "adjoint.hpp"
#include "kernels.hpp"
#include "lengths.hpp"
#include "plan.hpp"

namespace brahms {
namespace detail {

// One pass of a plan along `axis` with lines of length N1 N2; nl says where
// the RK4 step goes (NL_* of kernels.hpp); linear passes take one field per
// block.
template <int N1, int N2>
hipError_t launch_axis(int axis, int nl, int nf, const brahms_plan_s& p, PassArgs a);

// `count` steps of a plane wave (nt = N1 N2) from the row of a, and of a
// group of them from descriptors d.
template <int N1, int N2>
hipError_t launch_line_steps(const brahms_plan_s& p, const PassArgs& a, int count, bool merged, bool first);
template <int N1, int N2>
void launch_group_line_steps(int nf, unsigned m, hipStream_t st, const PassArgs* d, long long step, int count,
                             bool merged);

// One of the three passes of a long tau axis (sub-transforms N1 N2).
template <int N1, int N2, int AX>
hipError_t launch_long(int nl, int nf, const brahms_plan_s& p, PassArgs a);

// Geometry of a batch launch group: m problems of one shape and field count;
// wide: bits (x = 1, y = 2) of the axes whose linear passes run kWideBlock
// threads per block.
struct GroupGeom {
  unsigned m;
  int nx, ny, nt, nf;
  int wide;
};

// One pass over a launch group (descriptors d[m] of this step).
template <int N1, int N2>
void launch_group_pass(int axis, int nl, const GroupGeom& g, hipStream_t st, const PassArgs* d,
                       long long step);

// One of the three passes of a long tau axis over a launch group.
template <int N1, int N2, int AX>
void launch_group_long(int nl, const GroupGeom& g, hipStream_t st, const PassArgs* d, long long step);

// Blocks of an adjoint pass over `lines` lines of length n along axis.
inline int adjoint_blocks(int axis, long lines, int n) {
  const int n2 = kBlock / lines_per_block(n);
  const int lpb = split_threads(n2, axis) / n2;
  return int((lines + lpb - 1) / lpb);
}

// Whether a reverse pass of a plan along x or tau is better with the fields
// together in a thread (adjoint_pass_together) than with one field per thread:
// three fields, a launch that fills the chip, and room for three fields in a
// lane.  128^3: x, reverse half-step first, 45 against 56 us; tau, last, 42 /
// 64.  Not with 24 values of a field in a lane, where three of them leave one
// wave per SIMD (192 x 128 x 96, 16 steps: 4580 / 3694 us), nor in launches of
// few waves (narrow_launch; 128 x 128 x 64: 1990 / 1837).
inline bool adjoint_together(const brahms_plan_s& p, int axis) {
  const int n = axis == AX_X ? p.nx : p.nt, n2 = kBlock / lines_per_block(n);
  const long long lines = axis == AX_X ? (long long)p.ny * p.nt : (long long)p.nx * p.ny;
  return p.nf == 3 && n / n2 <= 16 && !narrow_launch(lines, n2);
}

// One adjoint pass (conj-propagator transforms with the RK4 half-step's VJP)
// along x or tau (VJP_* of adjoint.hpp; with VJP_TOGETHER where
// adjoint_together says so).
template <int N1, int N2>
void launch_adj_axis(int axis, int at, const brahms_plan_s& p, const AdjArgs& a);

}  // namespace detail
}  // namespace brahms
