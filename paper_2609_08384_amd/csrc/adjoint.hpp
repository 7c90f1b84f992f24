// Adjoint (reverse-mode) kernels of the chi(2) split-step z-loop (gfx950).
//
// Cotangents follow the convention g = dJ/dRe(A) + i dJ/dIm(A) for a real
// loss J, so that dJ = sum Re(conj(g) dA).  For a pointwise map
// A' = f(A, conj A) with dA' = M dA + B conj(dA) the cotangent of the input
// is g = M^H g' + B^T conj(g') (the transpose of the map seen as a real-linear
// map on (Re A, Im A)).
//
// * Linear step (Sec. 3.1): exp(L dz) = F^-1 diag(P) F is complex-linear, its
//   adjoint is F^-1 diag(conj P) F: the same axis passes with conjugated
//   propagators.
// * RK4 half-step (Sec. 3.1, coefficients as in rk4_point): reverse sweep over
//   the four stages, with the stage values recomputed in registers from the
//   half-step's input.  Every coefficient is w c_j(z) with
//   c_j = i kappa_j exp(i sigma_j Phi(z)), so d/dPhi of a term w c q is
//   i sigma_j w c q; the per-stage sums of Re(conj(g_term) i sigma_j term) over
//   the grid are dJ/dPhi at the stage positions z_a, z_a + h/2, z_a + h.
#pragma once

#include "kernels.hpp"

namespace brahms {

// g_y of the products Q (see chi2_products) for cotangent gq of Q.
template <int NF>
__device__ inline void chi2_products_vjp(const float2* y, const float2* gq, float2* gy) {
  if constexpr (NF == 3) {
    // Q_p = s i, Q_s = p conj(i), Q_i = p conj(s)
    gy[0] = cfma(cmul(y[2], gq[1]), y[1], gq[2]);
    gy[1] = cfmac(cmulc(gq[0], y[2]), y[0], gq[2]);
    gy[2] = cfmac(cmulc(gq[0], y[1]), y[0], gq[1]);
  } else {
    // Q_F = S conj(F), Q_S = F F
    const float2 t = cmulc(gq[1], y[0]);  // gS conj(F)
    const float2 u = cmulc(y[1], gq[0]);
    gy[0] = make_float2(fmaf(2.f, t.x, u.x), fmaf(2.f, t.y, u.y));
    gy[1] = cmul(y[0], gq[0]);
  }
}

// sum_j sigma_j Re(conj(g_j) i w_j) with w_j = c_j q_j
template <int NF>
__device__ inline float phase_term(const float2* g, const float2 (*co)[kNlCoef], int k,
                                   const float2* q, const float* sigma) {
  float s = 0.f;
#pragma unroll
  for (int j = 0; j < NF; ++j) {
    const float2 w = cmul(co[j][k], q[j]);
    // Re(conj(g) i w) = g.x * (-w.y) + g.y * w.x
    s = fmaf(sigma[j], fmaf(g[j].y, w.x, -(g[j].x * w.y)), s);
  }
  return s;
}

// Reverse sweep of one RK4 half-step at one grid point: y is the half-step's
// input, g holds the cotangent of its output on entry and of its input on
// exit; dphi[0..2] accumulate dJ/dPhi at z_a, z_a + h/2, z_a + h.
template <int NF>
__device__ inline void rk4_vjp_point(const float2* y, float2* g, const float2 (*co)[kNlCoef],
                                     const float* sigma, double* dphi) {
  float2 q1[NF], q2[NF], q3[NF], q4[NF], ys1[NF], ys2[NF], ys3[NF];
  chi2_products<NF>(y, q1);
#pragma unroll
  for (int j = 0; j < NF; ++j) ys1[j] = cfma(y[j], co[j][0], q1[j]);
  chi2_products<NF>(ys1, q2);
#pragma unroll
  for (int j = 0; j < NF; ++j) ys2[j] = cfma(y[j], co[j][1], q2[j]);
  chi2_products<NF>(ys2, q3);
#pragma unroll
  for (int j = 0; j < NF; ++j) ys3[j] = cfma(y[j], co[j][2], q3[j]);
  chi2_products<NF>(ys3, q4);

  float2 gout[NF], gq[NF], gys[NF], gy[NF];
#pragma unroll
  for (int j = 0; j < NF; ++j) gout[j] = g[j];
  // y' = y + b1 q1 + b2 q2 + b2 q3 + b4 q4, ys_k = y + a_k q_k
  float pa = phase_term<NF>(gout, co, 3, q1, sigma);
  float pm = phase_term<NF>(gout, co, 4, q2, sigma) + phase_term<NF>(gout, co, 4, q3, sigma);
  const float pe = phase_term<NF>(gout, co, 5, q4, sigma);
#pragma unroll
  for (int j = 0; j < NF; ++j) gq[j] = cmulc(gout[j], co[j][5]);        // conj(b4) g'
  chi2_products_vjp<NF>(ys3, gq, gys);                                   // g of ys3
  pm += phase_term<NF>(gys, co, 2, q3, sigma);
#pragma unroll
  for (int j = 0; j < NF; ++j) {
    gy[j] = cadd(gout[j], gys[j]);
    gq[j] = cfmac(cmulc(gys[j], co[j][2]), gout[j], co[j][4]);  // conj(a3) g_ys3 + conj(b2) g'
  }
  chi2_products_vjp<NF>(ys2, gq, gys);                                   // g of ys2
  pm += phase_term<NF>(gys, co, 1, q2, sigma);
#pragma unroll
  for (int j = 0; j < NF; ++j) {
    gy[j] = cadd(gy[j], gys[j]);
    gq[j] = cfmac(cmulc(gys[j], co[j][1]), gout[j], co[j][4]);  // conj(a2) g_ys2 + conj(b2) g'
  }
  chi2_products_vjp<NF>(ys1, gq, gys);                                   // g of ys1
  pa += phase_term<NF>(gys, co, 0, q1, sigma);
#pragma unroll
  for (int j = 0; j < NF; ++j) {
    gy[j] = cadd(gy[j], gys[j]);
    gq[j] = cfmac(cmulc(gys[j], co[j][0]), gout[j], co[j][3]);  // conj(a1) g_ys1 + conj(b1) g'
  }
  chi2_products_vjp<NF>(y, gq, gys);
#pragma unroll
  for (int j = 0; j < NF; ++j) g[j] = cadd(gy[j], gys[j]);
  dphi[0] += double(pa);
  dphi[1] += double(pm);
  dphi[2] += double(pe);
}

// ---------------------------------------------------------------------------
// Adjoint axis pass.  AT selects where the RK4 reverse sweep goes:
//   VJP_FIRST: the pass undoes the last pass of a forward step (whose RK4
//              half-step came after its transforms): reverse RK4 with the
//              saved half-step input, then FFT . conj(P) . IFFT;
//   VJP_LAST:  the pass undoes the first pass of a forward step: FFT .
//              conj(P) . IFFT, then reverse RK4 with the step's input;
//   VJP_PAIR:  VJP_LAST of step n, then VJP_FIRST of step n - 1, along the
//              same axis (the axes of a step's linear part commute, so the
//              reverse sweep takes them in an order of its own).
// g is updated in place; the block's dJ/dPhi partial sums (fixed-order
// reduction in double) go to dphi_out[block], three for each reverse RK4.
// ---------------------------------------------------------------------------
enum VjpWhere { VJP_FIRST = 1, VJP_LAST = 2, VJP_PAIR = 3 };
// Added to VJP_FIRST (x) or VJP_LAST (tau) for the launcher: the three fields
// together in a thread (adjoint_pass_together).
constexpr int VJP_TOGETHER = 4;

struct AdjArgs {
  float2* g[3];             // cotangent fields, in place
  const float2* y[3];       // saved input of the RK4 half-step
  const float2* tw;
  const float2* prop;
  const float2* nl;
  const DftConsts* consts;
  double* dphi_out;         // [gridDim.x][3]
  const float2* y2[3];      // VJP_PAIR: those of step n - 1's second half-step
  const float2* tw2;
  const float2* prop2;
  const float2* nl2;
  const DftConsts* consts2;
  double* dphi_out2;
  int nx, ny, nt;
  int slab;                 // as in PassArgs
  int axis_off, field_stride;
  float sigma[3];
};

// The block's three dJ/dPhi sums, in a fixed order: a tree within each of
// its groups of T threads, then the groups in turn.
template <int BLOCK, int T>
__device__ __forceinline__ void reduce_dphi(const double* dphi, double (*s_red)[BLOCK], double* out) {
  const int tid = threadIdx.x, g = tid % T;
#pragma unroll
  for (int k = 0; k < 3; ++k) s_red[k][tid] = dphi[k];
  __syncthreads();
  for (int w = T / 2; w > 0; w >>= 1) {
    if (g < w)
#pragma unroll
      for (int k = 0; k < 3; ++k) s_red[k][tid] += s_red[k][tid + w];
    __syncthreads();
  }
  if (tid < 3) {
    double s = 0.0;
#pragma unroll
    for (int i = 0; i < BLOCK / T; ++i) s += s_red[tid][i * T];
    out[blockIdx.x * 3 + tid] = s;
  }
}

// One field per thread (see axis_pass_split_body), the saved half-step inputs
// of a thread's points loaded with its cotangents; the reverse RK4 goes point
// by point (the asm ties: all points at once take 256 registers and leave one
// wave per SIMD).  Two fields at every size: with the saved states in memory
// (not in a cache) 128 x 128 x 64: x last 18.4 us (fields together: 26.4), x
// first 18.5 / 23.5, tau first 17.8 / 18.3; 128^3, x first 33.0 / 33.1, tau
// first 32.2 / 33.6.  What bounds it: six field transfers, 50 MB at 128 x 128 x
// 64, 10 us; the rest is the chain of two waves a SIMD.  A pair moves eight
// where two passes move twelve: 29-30 us against 19 + 20 (beside the next
// segment's forward steps on the other stream).  Three fields: where
// adjoint_together (launch.hpp) does not prefer the other form.
template <int N1, int N2, int AX, int NF, int AT>
__global__ __launch_bounds__((NF * split_threads(N2, AX))) void adjoint_pass(AdjArgs args) {
  constexpr int T = split_threads(N2, AX), BLOCK = NF * T;
  using G = LineGeom<N1, N2, T>;
  constexpr int N = G::N;
  constexpr bool WL = AX == AX_X && T == 64 && N2 <= 64 && 64 % N2 == 0;
  constexpr bool PAIR = AT == VJP_PAIR;
  // blocks of more than two waves per SIMD (three fields, 16 lanes on tau)
  // have 168 registers a lane: twiddles from LDS, and a pair's second states
  // loaded behind the first reverse RK4 rather than ahead of it
  constexpr bool TIGHT = BLOCK > 512;
  static_assert(AX == AX_X || AX == AX_T, "RK4 reverse sweeps live in the x or tau pass");
  constexpr int XS = N2 > 1 ? G::LDS_ELEMS : N1 * T;
  __shared__ float2 lds[NF * XS];
  __shared__ float2 s_tw[N], s_prop[NF * N], s_tw2[PAIR ? N : 1], s_prop2[PAIR ? NF * N : 1];
  __shared__ double s_red[3][BLOCK];

  const int tid = threadIdx.x;
  const int f = __builtin_amdgcn_readfirstlane(tid / T);
  const int g = tid % T;
  const int t = AX == AX_X ? g % N2 : g / G::LPB;
  const int li = AX == AX_X ? g / N2 : g % G::LPB;
  const unsigned bx = AX == AX_X ? slab_tile(args, blockIdx.x) : blockIdx.x;
  const LineAddr la = line_addr<AX, N>(args, bx * unsigned(G::LPB) + unsigned(li));
  const unsigned idx0 = la.base + unsigned(t) * la.estride;
  const unsigned field_bytes = unsigned(args.nx) * unsigned(args.ny) * unsigned(args.nt) * 8u;
  const unsigned lane_bytes = idx0 * 8u, slot_bytes = unsigned(N2) * la.estride * 8u;
  float2* mine = lds + f * XS;
  float2* lbuf = (N2 > 1) ? mine + li * G::LSTRIDE : mine;
  const DftConsts K = *args.consts;
  float2 co[NF][kNlCoef];
  load_coefficients<NF>(args.nl, co);
  float sigma[NF];
#pragma unroll
  for (int j = 0; j < NF; ++j) sigma[j] = args.sigma[j];

  constexpr int P = (N1 + NF - 1) / NF;
  auto load_points = [&](const float2* const* from, float2 (&y)[P][NF]) {
#pragma unroll
    for (int j = 0; j < NF; ++j) {
      const __amdgpu_buffer_rsrc_t ry = field_rsrc(from[j], field_bytes);
#pragma unroll
      for (int k = 0; k < P; ++k)
        y[k][j] = load_slot<false>(ry, lane_bytes, unsigned(min(f + NF * k, N1 - 1)) * slot_bytes);
    }
  };
  StageTables<N, NF, BLOCK, PAIR> st;
  st.begin(args, 0, tid);
  const __amdgpu_buffer_rsrc_t rg = field_rsrc(args.g[f], field_bytes);
  float2 v[N1];
#pragma unroll
  for (int e = 0; e < N1; ++e) v[e] = load_slot<false>(rg, lane_bytes, unsigned(e) * slot_bytes);
  float2 y[P][NF];
  load_points(args.y, y);
  st.end(false, tid, s_tw, s_prop, s_tw2, s_prop2);
  __syncthreads();  // s_tw, s_prop staged
  LaneTwiddles<N1, N2, !TIGHT> tw;
  tw.init(s_tw, t);

  float2 gg[P][NF];
  auto reverse_points = [&](float2 (&y)[P][NF], double (&dphi)[3]) {
    dphi[0] = dphi[1] = dphi[2] = 0.0;
#pragma unroll
    for (int k = 0; k < P; ++k) {
      if (N1 % NF == 0 || f + NF * k < N1) {
        // one point at a time: this point's values wait for the sums of the
        // previous one (an empty asm, no instructions)
#pragma unroll
        for (int j = 0; j < NF; ++j)
          asm volatile("" : "+v"(y[k][j].x), "+v"(y[k][j].y), "+v"(gg[k][j].x), "+v"(gg[k][j].y), "+v"(dphi[0]),
                            "+v"(dphi[1]), "+v"(dphi[2]));
        rk4_vjp_point<NF>(y[k], gg[k], co, sigma, dphi);
      }
    }
  };
  double dphi[3], dphi2[3];
  auto reverse_rk4 = [&]() {
    line_sync<WL>();   // this group's exchange rows are free
#pragma unroll
    for (int e = 0; e < N1; ++e) mine[e * T + g] = v[e];
    float2 yb[PAIR ? P : 1][NF];
    if constexpr (PAIR && !TIGHT) load_points(args.y2, yb);
    __syncthreads();
#pragma unroll
    for (int k = 0; k < P; ++k) {
      const int e = f + NF * k;
#pragma unroll
      for (int j = 0; j < NF; ++j)
        gg[k][j] = (N1 % NF == 0 || e < N1) ? lds[j * XS + e * T + g] : make_float2(0.f, 0.f);
    }
    reverse_points(y, dphi);
    if constexpr (PAIR) {
      if constexpr (TIGHT) {
        __builtin_amdgcn_sched_barrier(0);
        load_points(args.y2, yb);
      }
      load_coefficients<NF>(args.nl2, co);
      reverse_points(yb, dphi2);
    }
#pragma unroll
    for (int k = 0; k < P; ++k) {
      const int e = f + NF * k;
      if (N1 % NF == 0 || e < N1) {
#pragma unroll
        for (int j = 0; j < NF; ++j) lds[j * XS + e * T + g] = gg[k][j];
      }
    }
    __syncthreads();
#pragma unroll
    for (int e = 0; e < N1; ++e) v[e] = mine[e * T + g];
  };
  float2 (&v1)[1][N1] = reinterpret_cast<float2 (&)[1][N1]>(v);

  if constexpr (AT == VJP_FIRST) reverse_rk4();
  line_trip<N1, N2, 1, WL, true>(v1, tw, t, lbuf, s_prop + f * N, K);
  if constexpr (AT != VJP_FIRST) reverse_rk4();
  if constexpr (PAIR) {
    const DftConsts K2 = *args.consts2;
    tw.init(s_tw2, t);
    line_trip<N1, N2, 1, WL, true>(v1, tw, t, lbuf, s_prop2 + f * N, K2);
  }
  if (la.valid) {
#pragma unroll
    for (int e = 0; e < N1; ++e) store_slot<false>(rg, lane_bytes, unsigned(e) * slot_bytes, v[e]);
  } else {   // a line past the last one counts for nothing
    dphi[0] = dphi[1] = dphi[2] = 0.0;
    dphi2[0] = dphi2[1] = dphi2[2] = 0.0;
  }
  reduce_dphi<BLOCK, T>(dphi, s_red, args.dphi_out);
  if constexpr (PAIR) {
    __syncthreads();   // the sums are read
    reduce_dphi<BLOCK, T>(dphi2, s_red, args.dphi_out2);
  }
}

// Three fields, together in a thread: the reverse RK4 point by point on the
// thread's own values (no exchange between threads), the saved states read
// where they are used.  Only what adjoint_together takes: FIRST on x and LAST
// on tau (a step's axes commute, and these are the faster two), step by step
// rather than in pairs.  167-216 registers, two or three waves per SIMD; 18
// field transfers a step (with y) at 3.5 TB/s.  128^3, 20 steps: 4622 -> 4361
// us against pairs of one field per thread (recording beside), 256 x 128 x 128,
// 16 steps: 6050 -> 5566.
template <int N1, int N2, int AX, int AT>
__global__ __launch_bounds__(kBlock) void adjoint_pass_together(AdjArgs args) {
  constexpr int NF = 3;
  using G = LineGeom<N1, N2>;
  constexpr int N = G::N;
  constexpr bool WL = AX == AX_X && N2 <= 64 && 64 % N2 == 0;
  static_assert((AX == AX_X && AT == VJP_FIRST) || (AX == AX_T && AT == VJP_LAST), "x first, tau last");
  __shared__ float2 lds[G::LDS_ELEMS];
  __shared__ float2 s_tw[N], s_prop[NF * N];
  __shared__ double s_red[3][kBlock];

  const int tid = threadIdx.x;
  const int t = AX == AX_X ? tid % N2 : tid / G::LPB;
  const int li = AX == AX_X ? tid / N2 : tid % G::LPB;
  const unsigned bx = AX == AX_X ? slab_tile(args, blockIdx.x) : blockIdx.x;
  const LineAddr la = line_addr<AX, N>(args, bx * unsigned(G::LPB) + unsigned(li));
  const unsigned idx0 = la.base + unsigned(t) * la.estride;
  const unsigned field_bytes = unsigned(args.nx) * unsigned(args.ny) * unsigned(args.nt) * 8u;
  const unsigned lane_bytes = idx0 * 8u, slot_bytes = unsigned(N2) * la.estride * 8u;
  float2* lbuf = (N2 > 1) ? lds + li * G::LSTRIDE : lds;
  const DftConsts K = *args.consts;
  float2 co[NF][kNlCoef];
  load_coefficients<NF>(args.nl, co);
  float sigma[NF];
  __amdgpu_buffer_rsrc_t rg[NF], ry[NF];
#pragma unroll
  for (int j = 0; j < NF; ++j) {
    sigma[j] = args.sigma[j];
    rg[j] = field_rsrc(args.g[j], field_bytes);
    ry[j] = field_rsrc(args.y[j], field_bytes);
  }
  StageTables<N, NF, kBlock, false> st;
  st.begin(args, 0, tid);
  float2 v[NF][N1];
#pragma unroll
  for (int j = 0; j < NF; ++j)
#pragma unroll
    for (int e = 0; e < N1; ++e) v[j][e] = load_slot<false>(rg[j], lane_bytes, unsigned(e) * slot_bytes);
  st.end(false, tid, s_tw, s_prop, s_tw, s_prop);
  __syncthreads();  // s_tw, s_prop staged
  LaneTwiddles<N1, N2, false> tw;
  tw.init(s_tw, t);

  double dphi[3] = {0.0, 0.0, 0.0};
  auto reverse_rk4 = [&]() {
#pragma unroll
    for (int e = 0; e < N1; ++e) {
      float2 yy[NF], gg[NF];
#pragma unroll
      for (int j = 0; j < NF; ++j) {
        yy[j] = load_slot<false>(ry[j], lane_bytes, unsigned(e) * slot_bytes);
        gg[j] = v[j][e];
      }
      // one point at a time (an empty asm, no instructions)
#pragma unroll
      for (int j = 0; j < NF; ++j)
        asm volatile("" : "+v"(yy[j].x), "+v"(yy[j].y), "+v"(gg[j].x), "+v"(gg[j].y), "+v"(dphi[0]),
                          "+v"(dphi[1]), "+v"(dphi[2]));
      rk4_vjp_point<NF>(yy, gg, co, sigma, dphi);
#pragma unroll
      for (int j = 0; j < NF; ++j) v[j][e] = gg[j];
    }
  };
  if constexpr (AT == VJP_FIRST) reverse_rk4();
  line_trip<N1, N2, NF, WL, true>(v, tw, t, lbuf, s_prop, K);
  if (la.valid) {   // (the RK4 inside: it would be moved down to the stores, away from its states)
    if constexpr (AT == VJP_LAST) reverse_rk4();
#pragma unroll
    for (int j = 0; j < NF; ++j)
#pragma unroll
      for (int e = 0; e < N1; ++e) store_slot<false>(rg[j], lane_bytes, unsigned(e) * slot_bytes, v[j][e]);
  } else {   // a line past the last one counts for nothing
    dphi[0] = dphi[1] = dphi[2] = 0.0;
  }
  reduce_dphi<kBlock, kBlock>(dphi, s_red, args.dphi_out);
}

// Sum the per-block phase derivatives of a segment's adjoint passes (fixed
// order).  Block (i, w) handles step i of the segment and pass w (0: the
// reverse first half-step, 1: the reverse second half-step), which wrote
// parts[((i * 2 + w) * stride + b) * 3 + k] for its blocks b; out[6 i + 3 w +
// k] receives the sum over b (block size 256).  The axes may alternate: pass w
// has last_w blocks in the segment's last step and every second one before,
// other_w in those between.
static __global__ void reduce_dphi_segment(const double* parts, int last_0, int last_1, int other_0, int other_1,
                                           int stride, double* out) {
  __shared__ double s[256];
  const int i = blockIdx.x, w = blockIdx.y;
  const int nb = ((int(gridDim.x) - 1 - i) & 1) == 0 ? (w == 0 ? last_0 : last_1) : (w == 0 ? other_0 : other_1);
  const double* src = parts + (size_t(i) * 2 + w) * size_t(stride) * 3;
  for (int k = 0; k < 3; ++k) {
    double acc = 0.0;
    for (int b = threadIdx.x; b < nb; b += blockDim.x) acc += src[b * 3 + k];
    s[threadIdx.x] = acc;
    __syncthreads();
    for (int h = blockDim.x / 2; h > 0; h >>= 1) {
      if (threadIdx.x < h) s[threadIdx.x] += s[threadIdx.x + h];
      __syncthreads();
    }
    if (threadIdx.x == 0) out[6 * i + 3 * w + k] = s[0];
    __syncthreads();
  }
}

// dst = src over n complex values (checkpoint copies)
static __global__ void copy_field(float2* dst, const float2* src, long n) {
  long i = long(blockIdx.x) * blockDim.x + threadIdx.x;
  const long stride = long(gridDim.x) * blockDim.x;
  for (; i < n; i += stride) dst[i] = src[i];
}

static __global__ void zero_doubles(double* p, long n) {
  long i = long(blockIdx.x) * blockDim.x + threadIdx.x;
  const long stride = long(gridDim.x) * blockDim.x;
  for (; i < n; i += stride) p[i] = 0.0;
}

}  // namespace brahms
