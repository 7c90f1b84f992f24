// Definitions of the launchers declared in launch.hpp (included only by the
// per-length translation units len_*.hip, which instantiate them).
#pragma once

#include "launch.hpp"

namespace brahms {
namespace detail {

// ---------------------------------------------------------------------------
// plans: each supported axis length maps to a (N1, N2) split with N2 threads
// per line and N1 values per thread
// ---------------------------------------------------------------------------
inline unsigned blocks_of(long lines, int lpb) { return unsigned((lines + lpb - 1) / lpb); }

// A linear pass (one field per block) over `lines` lines along AX, with
// kBlock or (wide, where the split has a wide form) kWideBlock threads per
// block, or, in launches of few waves, with as few as split_threads, which
// spread over more CUs (two fields, 32^3: 2.8-3.1 instead of 3.3-3.6 us; 96 x
// 96 x 64, x: 8.4 / 9.9; CW 128 x 128: 3.7-4.0 / 4.8-4.9).
template <int N1, int N2, int AX>
void launch_linear(bool wide, long lines, int nf, hipStream_t st, PassArgs a) {
  if constexpr (wide_split<N1>()) {
    if (wide) {
      const dim3 grid(blocks_of(lines, LineGeom<N1, N2, kWideBlock>::LPB), 1, unsigned(nf));
      hipLaunchKernelGGL((axis_pass<N1, N2, AX, 1, NL_NONE, kWideBlock>), grid, dim3(kWideBlock), 0, st, a);
      return;
    }
  }
  constexpr int T = split_threads(N2, AX);
  if (T < kBlock && narrow_launch(lines * nf, N2)) {
    a.tiles = blocks_of(lines, T / N2);   // (the tau pass's tiles are its own blocks)
    a.tile_mul = 1;
    hipLaunchKernelGGL((axis_pass<N1, N2, AX, 1, NL_NONE, T>), dim3(a.tiles, 1, unsigned(nf)), dim3(T), 0, st, a);
    return;
  }
  const dim3 grid(blocks_of(lines, LineGeom<N1, N2>::LPB), 1, unsigned(nf));
  hipLaunchKernelGGL((axis_pass<N1, N2, AX, 1, NL_NONE>), grid, dim3(kBlock), 0, st, a);
}

template <int N1, int N2, int AX, int NF, int NL>
void launch_split(long lines, hipStream_t st, const PassArgs& a) {
  constexpr int T = split_threads(N2, AX);
  hipLaunchKernelGGL((axis_pass_split<N1, N2, AX, NF, NL>), dim3(blocks_of(lines, T / N2)), dim3(NF * T), 0, st, a);
}

// A pass with an RK4 step: the fields together in a thread, or one field per
// thread where the launch would leave SIMDs idle (narrow_launch; the same
// bits either way).
template <int N1, int N2, int AX, int NF, int NL>
void launch_rk4(long lines, hipStream_t st, const PassArgs& a) {
  if constexpr (together_split<N1>()) {
    if (!narrow_launch(lines, N2)) {
      hipLaunchKernelGGL((axis_pass<N1, N2, AX, NF, NL>), dim3(blocks_of(lines, LineGeom<N1, N2>::LPB)),
                         dim3(kBlock), 0, st, a);
      return;
    }
  }
  launch_split<N1, N2, AX, NF, NL>(lines, st, a);
}

// Half-step modes of x, y and tau passes: the transverse map runs on x and
// tau, both half-steps in one pass only on tau (plane waves).
template <int N1, int N2, int AX, int NF>
void launch_nl_nf(int nl, long lines, hipStream_t st, const PassArgs& a) {
  if (nl == (NL_AFTER | NL_FUSE)) return launch_rk4<N1, N2, AX, NF, NL_AFTER | NL_FUSE>(lines, st, a);
  if (nl == (NL_AFTER | NL_FUSE | NL_LIT))
    return launch_rk4<N1, N2, AX, NF, NL_AFTER | NL_FUSE | NL_LIT>(lines, st, a);
  if constexpr (AX != AX_Y) {
    if (nl == (NL_AFTER | NL_FUSE | NL_LIT | NL_MAP))
      return launch_rk4<N1, N2, AX, NF, NL_AFTER | NL_FUSE | NL_LIT | NL_MAP>(lines, st, a);
  }
  if constexpr (AX == AX_T) {
    if (nl == NL_BOTH) return launch_split<N1, N2, AX, NF, NL_BOTH>(lines, st, a);   // (one line)
  }
  if constexpr (AX != AX_Y) {
    if (nl == (NL_BEFORE | NL_MAP)) return launch_rk4<N1, N2, AX, NF, NL_BEFORE | NL_MAP>(lines, st, a);
    if (nl == (NL_AFTER | NL_MAP)) return launch_rk4<N1, N2, AX, NF, NL_AFTER | NL_MAP>(lines, st, a);
  }
  if (nl == NL_BEFORE) launch_rk4<N1, N2, AX, NF, NL_BEFORE>(lines, st, a);
  else launch_rk4<N1, N2, AX, NF, NL_AFTER>(lines, st, a);
}

template <int N1, int N2, int AX>
void launch_nl(int nf, int nl, long lines, hipStream_t st, const PassArgs& a) {
  if (nf == 3) launch_nl_nf<N1, N2, AX, 3>(nl, lines, st, a);
  else launch_nl_nf<N1, N2, AX, 2>(nl, lines, st, a);
}

template <int N1, int N2>
hipError_t launch_axis(int axis, int nl, int nf, const brahms_plan_s& p, PassArgs a) {
  a.tile_mul = 1;
  a.tiles = 1;
  const bool wide = wide_split<N1>() && ((p.wide >> axis) & 1) != 0;
  if (axis == AX_X) {
    const long lines = long(p.ny) * p.nt;
    if (nl == NL_NONE) launch_linear<N1, N2, AX_X>(wide, lines, nf, p.stream, a);
    else launch_nl<N1, N2, AX_X>(nf, nl, lines, p.stream, a);
  } else if (axis == AX_Y) {
    const long lines = long(p.nx) * p.nt;
    if (nl == NL_NONE) launch_linear<N1, N2, AX_Y>(wide, lines, nf, p.stream, a);
    else launch_nl<N1, N2, AX_Y>(nf, nl, lines, p.stream, a);
  } else {
    const long lines = long(p.nx) * p.ny;
    // linear tau passes (orders 2 and 3) take the tiles of their block size
    const int lpb = nl == NL_NONE && wide ? LineGeom<N1, N2, kWideBlock>::LPB : LineGeom<N1, N2>::LPB;
    a.tiles = blocks_of(lines, lpb);
    a.tile_mul = tile_multiplier(a.tiles);
    if (nl == NL_NONE) launch_linear<N1, N2, AX_T>(wide, lines, nf, p.stream, a);
    else launch_nl<N1, N2, AX_T>(nf, nl, lines, p.stream, a);
  }
  return hipGetLastError();
}

template <int N1, int N2>
hipError_t launch_line_steps(const brahms_plan_s& p, const PassArgs& a, int count, bool merged, bool first) {
  if (p.nf == 3)
    hipLaunchKernelGGL((line_steps<N1, N2, 3>), dim3(1), dim3(192), 0, p.stream, a, count, int(merged), int(first));
  else
    hipLaunchKernelGGL((line_steps<N1, N2, 2>), dim3(1), dim3(128), 0, p.stream, a, count, int(merged), int(first));
  return hipGetLastError();
}

template <int N1, int N2>
void launch_group_line_steps(int nf, unsigned m, hipStream_t st, const PassArgs* d, long long step, int count,
                             bool merged) {
  if (nf == 3)
    hipLaunchKernelGGL((line_steps_batched<N1, N2, 3>), dim3(m), dim3(192), 0, st, d, step, count, int(merged));
  else
    hipLaunchKernelGGL((line_steps_batched<N1, N2, 2>), dim3(m), dim3(128), 0, st, d, step, count, int(merged));
}

// The three passes of a long tau axis.  ONE: the plane is a multiple of a
// block's lines, so that a block's lines share the other index and need only
// N entries of the nt-point table instead of all of it (at nt = 1024, 8 KB
// for every 16 KB of field values, and 32 KB of LDS that keep blocks off the
// CU): 128 x 128 x 1024 and three fields, 193 / 181 / 193 -> 171 / 144 / 171
// us; 64 x 64 x 4096, 210 / 201 / 209 -> 167 / 156 / 167 us.
template <int N1, int N2, int AX, int NF, int NL>
void launch_long_pass(bool one, dim3 grid, hipStream_t st, const PassArgs& a) {
  if (one) hipLaunchKernelGGL((axis_pass<N1, N2, AX, NF, NL | NL_ONE>), grid, dim3(kBlock), 0, st, a);
  else hipLaunchKernelGGL((axis_pass<N1, N2, AX, NF, NL>), grid, dim3(kBlock), 0, st, a);
}

template <int N1, int N2, int AX>
hipError_t launch_long(int nl, int nf, const brahms_plan_s& p, PassArgs a) {
  constexpr int LPB = LineGeom<N1, N2>::LPB;
  a.tile_mul = 1;
  a.tiles = 1;
  const long plane = long(p.nx) * p.ny;
  const bool one = plane % LPB == 0;
  const unsigned blocks = blocks_of(plane * (p.nt / (N1 * N2)), LPB);
  if constexpr (AX == AX_TAI) {
    if (nl != NL_NONE) {   // the last pass of a step, with its second half-step
      const bool map = (nl & NL_MAP) != 0;
      if (nf == 3 && map) launch_long_pass<N1, N2, AX_TAI, 3, NL_AFTER | NL_MAP>(one, dim3(blocks), p.stream, a);
      else if (nf == 3) launch_long_pass<N1, N2, AX_TAI, 3, NL_AFTER>(one, dim3(blocks), p.stream, a);
      else if (map) launch_long_pass<N1, N2, AX_TAI, 2, NL_AFTER | NL_MAP>(one, dim3(blocks), p.stream, a);
      else launch_long_pass<N1, N2, AX_TAI, 2, NL_AFTER>(one, dim3(blocks), p.stream, a);
      return hipGetLastError();
    }
  }
  // linear passes (the inverse b pass too, when fused step pairs carry the
  // RK4 step on x and y): one field per block
  launch_long_pass<N1, N2, AX, 1, NL_NONE>(one, dim3(blocks, 1, unsigned(nf)), p.stream, a);
  return hipGetLastError();
}

// ---------------------------------------------------------------------------
// batches: the problem index is a grid dimension (blockIdx.y for passes over
// all fields, blockIdx.z / nf for passes of one field per block)
// ---------------------------------------------------------------------------
template <int N1, int N2, int AX, int BLOCK = kBlock>
void launch_batched_linear(long lines, const GroupGeom& g, hipStream_t st, const PassArgs* d, long long step) {
  const dim3 grid(blocks_of(lines, LineGeom<N1, N2, BLOCK>::LPB), 1, unsigned(g.nf) * g.m);
  hipLaunchKernelGGL((axis_pass_batched<N1, N2, AX, 1, NL_NONE, BLOCK>), grid, dim3(BLOCK), 0, st, d, step, g.nf);
}

// As launch_rk4, the lines of the whole group counted.
template <int N1, int N2, int AX, int NF, int NL>
void launch_batched_rk4(long lines, const GroupGeom& g, hipStream_t st, const PassArgs* d, long long step) {
  if constexpr (together_split<N1>()) {
    if (!narrow_launch((long long)lines * g.m, N2)) {
      hipLaunchKernelGGL((axis_pass_batched<N1, N2, AX, NF, NL>), dim3(blocks_of(lines, LineGeom<N1, N2>::LPB), g.m),
                         dim3(kBlock), 0, st, d, step, NF);
      return;
    }
  }
  constexpr int T = split_threads(N2, AX);
  hipLaunchKernelGGL((axis_pass_split_batched<N1, N2, AX, NF, NL>), dim3(blocks_of(lines, T / N2), g.m), dim3(NF * T),
                     0, st, d, step, NF);
}

template <int N1, int N2, int AX, int NF>
void launch_batched_nl_nf(int nl, long lines, const GroupGeom& g, hipStream_t st, const PassArgs* d, long long step) {
  if (nl == (NL_AFTER | NL_FUSE))
    return launch_batched_rk4<N1, N2, AX, NF, NL_AFTER | NL_FUSE>(lines, g, st, d, step);
  if (nl == (NL_AFTER | NL_FUSE | NL_LIT))
    return launch_batched_rk4<N1, N2, AX, NF, NL_AFTER | NL_FUSE | NL_LIT>(lines, g, st, d, step);
  if (nl == NL_BEFORE) launch_batched_rk4<N1, N2, AX, NF, NL_BEFORE>(lines, g, st, d, step);
  else launch_batched_rk4<N1, N2, AX, NF, NL_AFTER>(lines, g, st, d, step);
}

template <int N1, int N2, int AX>
void launch_batched_nl(int nl, long lines, const GroupGeom& g, hipStream_t st, const PassArgs* d, long long step) {
  if (g.nf == 3) launch_batched_nl_nf<N1, N2, AX, 3>(nl, lines, g, st, d, step);
  else launch_batched_nl_nf<N1, N2, AX, 2>(nl, lines, g, st, d, step);
}

// One axis of a group: its RK4 passes, its linear passes on kBlock threads
// and, for x and y, on kWideBlock threads.
template <int N1, int N2, int AX>
void launch_group_axis(int nl, long lines, const GroupGeom& g, hipStream_t st, const PassArgs* d, long long step) {
  if (nl != NL_NONE) return launch_batched_nl<N1, N2, AX>(nl, lines, g, st, d, step);
  if constexpr (AX != AX_T && wide_split<N1>()) {
    if ((g.wide >> AX) & 1) return launch_batched_linear<N1, N2, AX, kWideBlock>(lines, g, st, d, step);
  }
  // (a batch's linear tau passes keep the blocks of their descriptors' tiles)
  constexpr int T = split_threads(N2, AX);
  if constexpr (AX != AX_T && T < kBlock) {
    if (narrow_launch((long long)lines * g.nf * g.m, N2))
      return launch_batched_linear<N1, N2, AX, T>(lines, g, st, d, step);
  }
  launch_batched_linear<N1, N2, AX>(lines, g, st, d, step);
}

template <int N1, int N2>
void launch_group_pass(int axis, int nl, const GroupGeom& g, hipStream_t st, const PassArgs* d,
                       long long step) {
  if (axis == AX_X) launch_group_axis<N1, N2, AX_X>(nl, long(g.ny) * g.nt, g, st, d, step);
  else if (axis == AX_Y) launch_group_axis<N1, N2, AX_Y>(nl, long(g.nx) * g.nt, g, st, d, step);
  else launch_group_axis<N1, N2, AX_T>(nl, long(g.nx) * g.ny, g, st, d, step);
}

template <int N1, int N2, int AX, int NF, int NL>
void launch_group_long_pass(bool one, dim3 grid, const GroupGeom& g, hipStream_t st, const PassArgs* d,
                            long long step) {
  if (one)
    hipLaunchKernelGGL((axis_pass_batched<N1, N2, AX, NF, NL | NL_ONE>), grid, dim3(kBlock), 0, st, d, step, g.nf);
  else
    hipLaunchKernelGGL((axis_pass_batched<N1, N2, AX, NF, NL>), grid, dim3(kBlock), 0, st, d, step, g.nf);
}

template <int N1, int N2, int AX>
void launch_group_long(int nl, const GroupGeom& g, hipStream_t st, const PassArgs* d, long long step) {
  constexpr int LPB = LineGeom<N1, N2>::LPB;
  const long plane = long(g.nx) * g.ny;
  const bool one = plane % LPB == 0;
  const unsigned blocks = blocks_of(plane * (g.nt / (N1 * N2)), LPB);
  if constexpr (AX == AX_TAI) {   // (groups of long tau problems keep their five passes)
    if (g.nf == 3) launch_group_long_pass<N1, N2, AX_TAI, 3, NL_AFTER>(one, dim3(blocks, g.m), g, st, d, step);
    else launch_group_long_pass<N1, N2, AX_TAI, 2, NL_AFTER>(one, dim3(blocks, g.m), g, st, d, step);
  } else {
    launch_group_long_pass<N1, N2, AX, 1, NL_NONE>(one, dim3(blocks, 1, unsigned(g.nf) * g.m), g, st, d, step);
  }
}

// ---------------------------------------------------------------------------
// adjoint passes (x or tau, with the VJP of the half-step they undo)
// ---------------------------------------------------------------------------
// (the block counts are pass_blocks' and together_blocks' in adjoint.hip)
template <int AX>
long adjoint_lines(const brahms_plan_s& p) {
  return AX == AX_X ? long(p.ny) * p.nt : long(p.nx) * p.ny;
}

template <int N1, int N2, int AX, int NF, int AT>
void launch_adj(const brahms_plan_s& p, const AdjArgs& a) {
  constexpr int T = split_threads(N2, AX);
  hipLaunchKernelGGL((adjoint_pass<N1, N2, AX, NF, AT>), dim3(blocks_of(adjoint_lines<AX>(p), T / N2)), dim3(NF * T),
                     0, p.stream, a);
}

template <int N1, int N2, int AX, int NF>
void launch_adj_at(int at, const brahms_plan_s& p, const AdjArgs& a) {
  if constexpr (NF == 3 && N1 <= 16) {
    constexpr int AT = AX == AX_X ? VJP_FIRST : VJP_LAST;
    if (at == (AT | VJP_TOGETHER)) {
      hipLaunchKernelGGL((adjoint_pass_together<N1, N2, AX, AT>),
                         dim3(blocks_of(adjoint_lines<AX>(p), LineGeom<N1, N2>::LPB)), dim3(kBlock), 0, p.stream, a);
      return;
    }
  }
  if (at == VJP_PAIR) launch_adj<N1, N2, AX, NF, VJP_PAIR>(p, a);
  else if (at == VJP_FIRST) launch_adj<N1, N2, AX, NF, VJP_FIRST>(p, a);
  else launch_adj<N1, N2, AX, NF, VJP_LAST>(p, a);
}

template <int N1, int N2>
void launch_adj_axis(int axis, int at, const brahms_plan_s& p, const AdjArgs& a) {
  if (axis == AX_X) {
    if (p.nf == 3) launch_adj_at<N1, N2, AX_X, 3>(at, p, a);
    else launch_adj_at<N1, N2, AX_X, 2>(at, p, a);
  } else {
    if (p.nf == 3) launch_adj_at<N1, N2, AX_T, 3>(at, p, a);
    else launch_adj_at<N1, N2, AX_T, 2>(at, p, a);
  }
}

}  // namespace detail
}  // namespace brahms

// Explicit instantiations of the launchers of one line length (the adjoint
// takes the first split of a length only).
#define BRAHMS_INSTANTIATE_PASSES(N1, N2)                                                              \
  template hipError_t brahms::detail::launch_axis<N1, N2>(int, int, int, const brahms_plan_s&,        \
                                                          brahms::PassArgs);                           \
  template void brahms::detail::launch_group_pass<N1, N2>(int, int, const brahms::detail::GroupGeom&, \
                                                          hipStream_t, const brahms::PassArgs*,        \
                                                          long long);                                  \
  template hipError_t brahms::detail::launch_line_steps<N1, N2>(const brahms_plan_s&,                 \
                                                                const brahms::PassArgs&, int, bool,   \
                                                                bool);                                \
  template void brahms::detail::launch_group_line_steps<N1, N2>(int, unsigned, hipStream_t,           \
                                                                const brahms::PassArgs*, long long,   \
                                                                int, bool);

#define BRAHMS_INSTANTIATE_LENGTH(N1, N2)                                                              \
  BRAHMS_INSTANTIATE_PASSES(N1, N2)                                                                    \
  template void brahms::detail::launch_adj_axis<N1, N2>(int, int, const brahms_plan_s&,               \
                                                        const brahms::AdjArgs&);

// Explicit instantiations of the three long-tau passes of one sub-length.
#define BRAHMS_INSTANTIATE_LONG_AX(N1, N2, AX)                                                          \
  template hipError_t brahms::detail::launch_long<N1, N2, AX>(int, int, const brahms_plan_s&,          \
                                                              brahms::PassArgs);                        \
  template void brahms::detail::launch_group_long<N1, N2, AX>(int, const brahms::detail::GroupGeom&,   \
                                                              hipStream_t, const brahms::PassArgs*,     \
                                                              long long);
#define BRAHMS_INSTANTIATE_LONG(N, N1, N2)            \
  BRAHMS_INSTANTIATE_LONG_AX(N1, N2, brahms::AX_TAF) \
  BRAHMS_INSTANTIATE_LONG_AX(N1, N2, brahms::AX_TB)  \
  BRAHMS_INSTANTIATE_LONG_AX(N1, N2, brahms::AX_TAI)
