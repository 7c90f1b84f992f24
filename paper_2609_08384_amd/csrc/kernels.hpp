// Device kernels of the chi(2) split-step z-loop (gfx950).
//
// One z-step (symmetric splitting N/2 - L - N/2, Sec. 3.1 eq. expon) is made
// of three passes over the fields, each a batch of independent 1D lines:
//
//   X pass : RK4 half-step of the coupled chi(2) equations (eqs. CEp/CEs/CEi),
//            then FFT_x . P_x . IFFT_x                    (all fields together)
//   Y pass : FFT_y . P_y . IFFT_y                          (one field per block)
//   T pass : FFT_tau . P_tau . IFFT_tau, then the second RK4 half-step
//
// The linear step exp(L dz) is separable, L = L_x + L_y + L_tau with the
// three parts acting on different axes, so its Fourier-space form is the
// product of three commuting 1D transform-multiply-inverse operators; this is
// the paper's own split into a tau step and an xy step (Sec. 4.3), taken one
// axis further.  Fields stay x-fastest, [nt][ny][nx] complex64, in place:
// the y and tau passes read their lines with a stride instead of
// materialising the paper's reordered copy.  The passes may run in either
// order (x, y, tau or tau, y, x); a tau axis longer than 256 takes three
// passes (a four-step transform, AX_TAF / AX_TB / AX_TAI below).  Where two
// consecutive steps meet along one axis, the one's T pass and the other's X
// pass (or the other way round) are a single fused pass, NL_FUSE: two reads
// and writes of the fields per step.
#pragma once

#include <hip/hip_runtime.h>

#include "dft.hpp"

namespace brahms {

constexpr int kBlock = 256;        // threads per block in every pass but the wide linear ones
constexpr int kNlCoef = 6;         // RK4 coefficients per field per half-step

enum Axis { AX_X = 0, AX_Y = 1, AX_T = 2,
            // a tau axis longer than one line transform, nt = A B, tau = a + A b
            // (a four-step transform over three passes):
            AX_TAF = 3,   // B-point transforms over b, times exp(-2 pi i a k_b / nt)
            AX_TB = 4,    // A-point transforms over a, propagator, inverse transforms
            AX_TAI = 5 }; // times exp(+2 pi i a k_b / nt), inverse B-point transforms
constexpr int kMaxLongT = 4096;   // longest tau axis (entries of the staged table)

__host__ __device__ constexpr bool long_tau_kind(int ax) { return ax >= AX_TAF; }
enum NlMode { NL_NONE = 0, NL_BEFORE = 1, NL_AFTER = 2,
              NL_BOTH = 3 };   // both half-steps in one pass (the only pass of a step)
// Added to NL_BEFORE / NL_AFTER: the mismatch phase also has a transverse
// part (a per-(x, y) table of exp(i m(x, y) Psi(z)) for each RK4 stage).
constexpr int NL_MAP = 4;
// Added to NL_AFTER (fused step pair): after the RK4 step the pass applies
// the next z-step's transform along the same axis, with that step's tables
// (tw2, prop2, consts2), so the last axis of step n and the first axis of
// step n + 1 cost one read and one write of the fields.
constexpr int NL_FUSE = 8;
// Added to NL_AFTER | NL_FUSE (literal half-steps): the second half-step of
// step n and the first one of step n + 1 instead of one RK4 step over both.
constexpr int NL_LIT = 16;
// Added to a long tau pass whose blocks each hold lines of one value of the
// other index (a or k_b): the plane is a multiple of a block's lines.
constexpr int NL_ONE = 32;

struct PassArgs {
  float2* f[3];          // fields read (complex64, [nt][ny][nx])
  float2* fo[3];         // fields written (== f for an in-place pass)
  float2* pre[3];        // if pre[0]: the last pass also stores its values
                         // just before the RK4 half-step here
  int conj;              // multiply by conj(P) (adjoint linear step)
  int slab;              // x and y passes: tiles in slabs (slab_tile)
  const float2* tw;      // this step's forward twiddles exp(-2 pi i m / N), m < N
  const float2* prop;    // this step's propagators, field j's table of this
                         // axis at prop + j * field_stride + axis_off
  const float2* nl;      // RK4 coefficients of the step's first half-step (NL_LIT:
                         // of the next step's), [nf][6]
  const float2* nl2;     // those of its second half-step (or, when adjacent
                         // halves are merged, of one RK4 step of size dz
                         // from z_n + dz/2)
  const DftConsts* consts;  // this step's register-DFT constants
  int nx, ny, nt;
  int axis_off, field_stride;
  unsigned tile_mul;     // block -> tile map: tile = (block * tile_mul) mod tiles
  unsigned tiles;        // number of tiles (blocks along x of the launch)
  long long nz;          // batched launches: the instance is done once step >= nz
  const float2* map;     // NL_MAP: exp(i m(x,y) Psi) at this half-step's three
                         // stage positions, [3][ny][nx]
  const float2* tw2;     // NL_FUSE: the next step's twiddles, propagators and
  const float2* prop2;   // DFT constants along the same axis
  const DftConsts* consts2;
  const float2* map2;    // NL_LIT with NL_MAP: map of the next step's first half-step
};

// ---------------------------------------------------------------------------
// chi(2) RK4 point update.  With c_j(z) = i kappa_j exp(sigma_j i Phi(z)) and
// the bilinear products Q_j (p: s i, s: p i*, i: p s*; SHG F: S F*, S: F F)
// one classical RK4 step of size h from z_a is
//   y2 = y + a1 Q(y),  y3 = y + a2 Q(y2),  y4 = y + a3 Q(y3),
//   y' = y + b1 Q(y) + b2 Q(y2) + b2 Q(y3) + b4 Q(y4)
// with a1 = h/2 c(z_a), a2 = h/2 c(z_m), a3 = h c(z_m), b1 = h/6 c(z_a),
// b2 = h/3 c(z_m), b4 = h/6 c(z_a + h), z_m = z_a + h/2.  The coefficients
// are formed in double precision per half-step by the table kernel.
// Adjacent halves (the second half of step n and the first of step n + 1)
// may be merged into one RK4 step of size h = dz from z_n + dz/2: the exact
// flows compose, and the two integrators differ by O(h^5) per step.
// ---------------------------------------------------------------------------
template <int NF>
__device__ inline void chi2_products(const float2* y, float2* q) {
  if constexpr (NF == 3) {
    q[0] = cmul(y[1], y[2]);
    q[1] = cmulc(y[0], y[2]);
    q[2] = cmulc(y[0], y[1]);
  } else {
    q[0] = cmulc(y[1], y[0]);
    q[1] = cmul(y[0], y[0]);
  }
}

__device__ inline float2 cfma(float2 acc, float2 c, float2 q) {  // acc + c q
  return make_float2(fmaf(c.x, q.x, fmaf(-c.y, q.y, acc.x)),
                     fmaf(c.x, q.y, fmaf(c.y, q.x, acc.y)));
}

__device__ inline float2 cfmac(float2 acc, float2 a, float2 b) {  // acc + a conj(b)
  return make_float2(fmaf(a.x, b.x, fmaf(a.y, b.y, acc.x)),
                     fmaf(a.y, b.x, fmaf(-a.x, b.y, acc.y)));
}

// A value that is the same in every lane, moved into scalar registers.
__device__ inline float2 wave_uniform(float2 v) {
  return make_float2(__int_as_float(__builtin_amdgcn_readfirstlane(__float_as_int(v.x))),
                     __int_as_float(__builtin_amdgcn_readfirstlane(__float_as_int(v.y))));
}

// Transverse part of the mismatch phase at one stage: Q_j times
// exp(i sigma_j m Psi) = w (sigma = +1) or conj(w) (sigma = -1, the
// sum-frequency field: p of three fields, S of SHG).
template <int NF>
__device__ inline void rotate_products(float2* q, float2 w) {
  constexpr int neg = NF == 3 ? 0 : 1;
#pragma unroll
  for (int j = 0; j < NF; ++j) q[j] = j == neg ? cmulc(q[j], w) : cmul(q[j], w);
}

// MAP: w[0], w[1], w[2] are the transverse phase factors at z_a, z_a + h/2
// and z_a + h (unused otherwise).
//
// The update sums stage values rather than increments: a1 = 3 b1, a2 = 3 b2 / 2
// and a3 = 3 b2, so b1 Q(y) = (y2 - y) / 3, b2 Q(y2) = 2 (y3 - y) / 3 and
// b2 Q(y3) = (y4 - y) / 3, and
//   y' = y + (y2 + 2 y3 + y4 - 4 y) / 3 + b4 Q(y4).
// Two operations per stage and field replace the complex multiply-add of
// each increment.  The factor 1/3 (rounded to FP32) scales only the O(h)
// bracket, so its rounding biases the nonlinear increment by ~3e-8 of itself
// and never the field; the bracket's rounding errors are of the size of the
// increment sums' (about one ulp of y per step) and independent from step to
// step.
template <int NF, bool MAP = false>
__device__ inline void rk4_point(float2* y, const float2 (*co)[kNlCoef], const float2* w = nullptr) {
  constexpr float kThird = 1.0f / 3.0f;
  float2 q[NF], s[NF], ys[NF];
  chi2_products<NF>(y, q);
  if constexpr (MAP) rotate_products<NF>(q, w[0]);
#pragma unroll
  for (int j = 0; j < NF; ++j) {
    ys[j] = cfma(y[j], co[j][0], q[j]);   // y2
    s[j] = ys[j];
  }
  chi2_products<NF>(ys, q);
  if constexpr (MAP) rotate_products<NF>(q, w[1]);
#pragma unroll
  for (int j = 0; j < NF; ++j) {
    ys[j] = cfma(y[j], co[j][1], q[j]);   // y3
    s[j] = make_float2(fmaf(2.0f, ys[j].x, s[j].x), fmaf(2.0f, ys[j].y, s[j].y));
  }
  chi2_products<NF>(ys, q);
  if constexpr (MAP) rotate_products<NF>(q, w[1]);
#pragma unroll
  for (int j = 0; j < NF; ++j) {
    ys[j] = cfma(y[j], co[j][2], q[j]);   // y4
    s[j] = cadd(s[j], ys[j]);
  }
  chi2_products<NF>(ys, q);
  if constexpr (MAP) rotate_products<NF>(q, w[2]);
#pragma unroll
  for (int j = 0; j < NF; ++j) {
    const float2 d = make_float2(fmaf(-4.0f, y[j].x, s[j].x), fmaf(-4.0f, y[j].y, s[j].y));
    const float2 u = make_float2(fmaf(kThird, d.x, y[j].x), fmaf(kThird, d.y, y[j].y));
    y[j] = cfma(u, co[j][5], q[j]);
  }
}

// ---------------------------------------------------------------------------
// One line transform of length N = N1 N2 (N2 divides N1) by N2 threads.
// Thread t holds x[t + N2 e] in slot e (e < N1).  Stage 1: an N1-point DFT in
// registers over e, times exp(-+2 pi i t k1 / N).  Exchange through LDS.
// Stage 2: for each k1 = t + N2 a, an N2-point DFT over the N2 threads' values.
// The result X[k1 + N1 k2] lands in slot a + (N1/N2) k2, i.e. thread t again
// holds index t + N2 e in slot e, so the inverse transform starts from the
// same layout without another exchange.
// ---------------------------------------------------------------------------
template <int N1, int N2, int BLOCK = kBlock>
struct LineGeom {
  static constexpr int N = N1 * N2;
  static constexpr int LPB = BLOCK / N2;                   // lines per block
  static constexpr int ROW = (N2 > 1) ? N2 + 1 : 1;        // padded LDS row
  static constexpr int LS0 = N1 * ROW;
  static constexpr int LSTRIDE = (N2 > 1) ? (LS0 | 1) : LS0;  // odd stride
  static constexpr int LDS_ELEMS = (N2 > 1) ? LPB * LSTRIDE : 1;
};

// Synchronisation of a line's lanes around its LDS exchange: the block's
// barrier, or, when every line lies within one wavefront (WAVE), only an
// ordering fence (a wave's LDS instructions complete in issue order).
template <bool WAVE>
__device__ __forceinline__ void line_sync() {
  if constexpr (WAVE) {
    __builtin_amdgcn_fence(__ATOMIC_SEQ_CST, "wavefront");
    __builtin_amdgcn_wave_barrier();
    __builtin_amdgcn_fence(__ATOMIC_SEQ_CST, "wavefront");
  } else {
    __syncthreads();
  }
}

// The lane's inter-stage twiddles exp(-2 pi i t k1 / N): kept in registers
// for a whole pass (REG: the 2 N1 values are then read from LDS once instead
// of once per field and direction), or read where they are used.
template <int N1, int N2, bool REG>
struct LaneTwiddles {
  float2 w[REG ? N1 : 1];
  const float2* tw;
  int t;
  __device__ __forceinline__ void init(const float2* table, int lane) {
    tw = table;
    t = lane;
    if constexpr (REG && N2 > 1) {
#pragma unroll
      for (int k1 = 1; k1 < N1; ++k1) w[k1] = tw[t * k1];
    }
  }
  __device__ __forceinline__ float2 at(int k1) const {
    if constexpr (REG) return w[k1];
    else return tw[t * k1];
  }
};

// Stage 1 of a transform: the N1-point DFT and the inter-stage twiddles.
template <int N1, int N2, bool INV, bool REG>
__device__ __forceinline__ void line_stage1(float2 (&v)[N1], const LaneTwiddles<N1, N2, REG>& tw,
                                            const DftConsts& K) {
  dft<N1, INV>(v, K);
  if constexpr (N2 > 1) {
#pragma unroll
    for (int k1 = 1; k1 < N1; ++k1) v[k1] = INV ? cmulc(v[k1], tw.at(k1)) : cmul(v[k1], tw.at(k1));
  }
}

// Stage 2, on the values of exchange_get: v[a N2 + n2] -> slot a + (N1/N2) k2.
template <int N1, int N2, bool INV>
__device__ __forceinline__ void line_stage2(float2 (&v)[N1], const DftConsts& K) {
  if constexpr (N2 > 1) {
    constexpr int R = N1 / N2;
    float2 o[N1];
#pragma unroll
    for (int a = 0; a < R; ++a) {
      float2 u[N2];
#pragma unroll
      for (int n2 = 0; n2 < N2; ++n2) u[n2] = v[a * N2 + n2];
      dft<N2, INV>(u, K);
#pragma unroll
      for (int k2 = 0; k2 < N2; ++k2) o[a + R * k2] = u[k2];
    }
#pragma unroll
    for (int e = 0; e < N1; ++e) v[e] = o[e];
  }
}

// The exchange between the stages through the line's LDS row.
template <int N1, int N2, bool WAVE>
__device__ __forceinline__ void exchange(float2 (&v)[N1], int t, float2* lbuf) {
  if constexpr (N2 > 1) {
    using G = LineGeom<N1, N2>;
    constexpr int R = N1 / N2;
    line_sync<WAVE>();  // earlier readers of this line's LDS row are done
#pragma unroll
    for (int k1 = 0; k1 < N1; ++k1) lbuf[k1 * G::ROW + t] = v[k1];
    line_sync<WAVE>();
#pragma unroll
    for (int a = 0; a < R; ++a)
#pragma unroll
      for (int n2 = 0; n2 < N2; ++n2) v[a * N2 + n2] = lbuf[(t + N2 * a) * G::ROW + n2];
    // the reads are issued here: what follows in the source runs while they
    // are under way
    __builtin_amdgcn_sched_barrier(0);
  }
}

// One whole transform.
template <int N1, int N2, bool INV, bool WAVE, bool REG>
__device__ __forceinline__ void line_fft(float2 (&v)[N1], const LaneTwiddles<N1, N2, REG>& tw, int t, float2* lbuf,
                                         const DftConsts& K) {
  line_stage1<N1, N2, INV>(v, tw, K);
  exchange<N1, N2, WAVE>(v, t, lbuf);
  line_stage2<N1, N2, INV>(v, K);
}

// FFT . P . IFFT along the line for the NF fields a lane holds (prop: P of
// field j at prop + j N; CONJ: conj(P)).  The fields' transforms are
// interleaved: while one field's exchange is under way (its LDS reads take
// some hundred cycles, and a SIMD holds three waves at most here) the lane
// works on the registers of another.  With the twiddles in registers this
// took the fused x / tau passes of 256^3 points and three fields from 196 /
// 219 us to 181 / 200 us, and those of 64^3 points and two fields from 8.7 /
// 9.1 us to 7.9 / 8.3 us (one field after another, twiddles from LDS).
template <int N1, int N2, int NF, bool WAVE, bool CONJ, bool REG>
__device__ __forceinline__ void line_trip(float2 (&v)[NF][N1], const LaneTwiddles<N1, N2, REG>& tw, int t,
                                          float2* lbuf, const float2* prop, const DftConsts& K) {
  auto middle = [&](int j) {   // the forward transform's end, P, the inverse one's beginning
    line_stage2<N1, N2, false>(v[j], K);
#pragma unroll
    for (int e = 0; e < N1; ++e) {
      const float2 p = prop[j * N1 * N2 + t + N2 * e];
      v[j][e] = CONJ ? cmulc(v[j][e], p) : cmul(v[j][e], p);
    }
    line_stage1<N1, N2, true>(v[j], tw, K);
  };
  if constexpr (N2 == 1) {   // nothing to wait for: one field after another
#pragma unroll
    for (int j = 0; j < NF; ++j) {
      line_stage1<N1, N2, false>(v[j], tw, K);
      middle(j);
      if (j + 1 < NF) {   // (the next field begins behind this one's results: no instructions)
#pragma unroll
        for (int e = 0; e < N1; ++e)
          asm volatile("" : "+v"(v[j][e].x), "+v"(v[j][e].y), "+v"(v[j + 1][e].x), "+v"(v[j + 1][e].y));
      }
    }
    return;
  }
  // (the schedule barriers keep the pieces apart: their temporaries would
  // not all fit beside the fields' registers)
  line_stage1<N1, N2, false>(v[0], tw, K);
#pragma unroll
  for (int j = 0; j < NF; ++j) {
    exchange<N1, N2, WAVE>(v[j], t, lbuf);
    if (j + 1 < NF) line_stage1<N1, N2, false>(v[j + 1], tw, K);
    __builtin_amdgcn_sched_barrier(0);
    if (j > 0) middle(j - 1);
  }
#pragma unroll
  for (int j = 0; j < NF; ++j) {
    if (j == 0 && NF == 1) middle(0);
    exchange<N1, N2, WAVE>(v[j], t, lbuf);
    if (j == 0 && NF > 1) middle(NF - 1);
    __builtin_amdgcn_sched_barrier(0);
    if (j > 0) line_stage2<N1, N2, true>(v[j - 1], K);
  }
  line_stage2<N1, N2, true>(v[NF - 1], K);
}

// ---------------------------------------------------------------------------
// Field access.  Field values are streamed once per pass; the addresses are a
// uniform base (scalar registers) plus a 32-bit element offset.
// ---------------------------------------------------------------------------
#ifndef BRAHMS_NT_X
#define BRAHMS_NT_X 1
#endif
#ifndef BRAHMS_NT_YT
#define BRAHMS_NT_YT 0
#endif
// Blocks of kBlock threads per CU the pass kernels are compiled for: 3 is
// 3 waves per SIMD, a budget of 168 VGPRs (granules of 8 out of 512).  The
// three-field passes that carry an RK4 step take 162-168 with 16 values a
// lane (a batch's keep one or two values in scratch memory, those of 24
// values up to six) and the fused
// step-pair pass's LDS allows 3 blocks as well; without the bound the
// compiler may take more registers and leave room for 2 waves only, which
// cost the fused pass ~15 % of its speed.  Kernels whose LDS already limits
// them to fewer blocks keep their register count.  Lines of 18 and 24 values
// per lane are compiled for two blocks, linear passes of 36 for one.
#ifndef BRAHMS_MIN_BLOCKS
#define BRAHMS_MIN_BLOCKS 3
#endif

typedef float f32x2 __attribute__((ext_vector_type(2)));

// Tie a point's RK4 inputs to the previous point's results with an empty asm
// (no instructions): the points of a thread are then updated one after the
// other instead of all interleaved, which would run out of registers.
template <int NF, int N1>
__device__ __forceinline__ void point_link(float2* y, float2 (&v)[NF][N1], int prev) {
#pragma unroll
  for (int j = 0; j < NF; ++j)
    asm volatile("" : "+v"(y[j].x), "+v"(y[j].y), "+v"(v[j][prev].x), "+v"(v[j][prev].y));
}

// The fields of a pass are read and written through buffer resources: the
// field's base and byte size sit in scalar registers, a lane's slot e at the
// lane's byte offset plus the uniform offset 8 e estep, which the scalar unit
// forms, so the slots' addresses take no vector instructions (global
// addressing takes a 64-bit add per slot).  The byte offsets fit 32 bits:
// a field holds at most 2^28 values.  Accesses past the size read zero and
// store nothing.
constexpr int kRsrcWord3 = 0x00020000;   // raw, untyped 32-bit buffer

__device__ inline __amdgpu_buffer_rsrc_t field_rsrc(const float2* base, unsigned bytes) {
  return __builtin_amdgcn_make_buffer_rsrc(const_cast<float2*>(base), short(0), int(bytes), kRsrcWord3);
}

template <bool NT>
__device__ inline float2 load_slot(__amdgpu_buffer_rsrc_t r, unsigned lane_bytes, unsigned slot_bytes) {
  const f32x2 v = __builtin_amdgcn_raw_buffer_load_b64(r, lane_bytes, slot_bytes, NT ? 2 : 0);
  return make_float2(v.x, v.y);
}

template <bool NT>
__device__ inline void store_slot(__amdgpu_buffer_rsrc_t r, unsigned lane_bytes, unsigned slot_bytes,
                                  float2 v) {
  f32x2 w;
  w.x = v.x;
  w.y = v.y;
  __builtin_amdgcn_raw_buffer_store_b64(w, r, lane_bytes, slot_bytes, NT ? 2 : 0);
}

// Transverse phase factors at a half-step's three stage positions for the
// (x, y) at the lane's byte offset plus the uniform slot_bytes, through a
// buffer resource as the fields are: with 64-bit addresses of its own each of
// the three factors of every slot along x takes two registers, and with three
// fields 44-58 of a lane's values went to scratch memory.
__device__ __forceinline__ void map_factors(__amdgpu_buffer_rsrc_t map, unsigned plane, unsigned lane_bytes,
                                            unsigned slot_bytes, float2* w) {
#pragma unroll
  for (int k = 0; k < 3; ++k) w[k] = load_slot<false>(map, lane_bytes, unsigned(k) * plane * 8u + slot_bytes);
}

// ---------------------------------------------------------------------------
// The fused axis pass.  AX selects the line family:
//   X: line = (y, tau), element stride 1, lanes t-fastest (contiguous loads)
//   Y: line = (x, tau), element stride nx, lanes x-fastest (coalesced rows)
//   T: line = (x, y),   element stride nx*ny, lanes (x,y)-fastest
// NF is the number of fields held by one thread (Y: 1, one field per block).
// ---------------------------------------------------------------------------
// Where a line's elements lie.  Lines past the last one (the last block's)
// are given the last line's addresses: they read and compute like it and
// store nothing (valid is false).
struct LineAddr {
  unsigned base, estride;
  unsigned lidx;   // long tau axis: a (b passes) or k_b (a pass) of the line
  bool valid;
};

template <int AX, int N, class Args>
__device__ __forceinline__ LineAddr line_addr(const Args& args, unsigned line) {
  const unsigned nx = args.nx, plane = unsigned(args.nx) * unsigned(args.ny);
  LineAddr a{0, 1, 0, true};
  if constexpr (AX == AX_X) {
    const unsigned lines = unsigned(args.ny) * unsigned(args.nt);
    a.valid = line < lines;
    a.base = min(line, lines - 1u) * nx;
  } else if constexpr (AX == AX_Y) {
    // lines (x, tau) numbered x-fastest, so that a block's lines are
    // consecutive x (coalesced rows) and only the last block can be partial
    const unsigned lines = nx * unsigned(args.nt);
    a.valid = line < lines;
    line = min(line, lines - 1u);
    a.base = line % nx + plane * (line / nx);
    a.estride = nx;
  } else if constexpr (long_tau_kind(AX)) {
    // lines (column, a) of the b transforms or (column, k_b) of the a
    // transforms, column-fastest: a block's lines are consecutive columns
    const unsigned nsub = unsigned(args.nt) / unsigned(N);     // A (b passes) or B (a pass)
    a.valid = line < plane * nsub;
    line = min(line, plane * nsub - 1u);
    const unsigned col = line % plane;
    a.lidx = line / plane;
    if constexpr (AX == AX_TB) {
      a.base = col + plane * unsigned(N) * a.lidx;   // elements a at tau = a + A k_b
      a.estride = plane;
    } else {
      a.base = col + plane * a.lidx;                 // elements b at tau = a + A b
      a.estride = plane * nsub;
    }
  } else {
    a.valid = line < plane;
    a.base = min(line, plane - 1u);
    a.estride = plane;
  }
  return a;
}

// This step's twiddles and the block's propagators go through LDS, the
// fields straight to registers.  All table loads are issued first and
// together (begin), then the field loads; only then are the table values
// waited for (loads return in order) and written to LDS (end), with the
// field loads still in flight: one memory latency instead of one per table
// and loop trip, and no block that waits for its tables with no field load
// outstanding (long tau passes of 128 x 128 x 1024: 11 % less time for the
// whole step).  WRAP (a plan's linear passes of kBlock threads): threads past a
// table's end take its entries once more, the same values to the same places.  Where their writes
// are left out, the compiler moves the loads down into the branch, behind the
// fields': linear passes of 128^3 points and two fields 17.1 -> 19.6 us in x,
// 12.3 -> 13.7 in tau.  Passes with an RK4 step and batches, whose waves hide
// that, lose 1-2 % by the added loads (16 problems of 64^3: 928 / 947), and so
// do blocks of 512 threads (128^3, three fields: 1674 / 1717 a run).
template <int N, int NF, int BLOCK, bool FUSE, bool WRAP = false>
struct StageTables {
  static constexpr int TT = (N + BLOCK - 1) / BLOCK;        // table entries per thread
  static constexpr int TP = (NF * N + BLOCK - 1) / BLOCK;
  float2 tw[TT], prop[TP], tw2[FUSE ? TT : 1], prop2[FUSE ? TP : 1];

  template <int SIZE>   // the table entry of a thread in round q
  __device__ static __forceinline__ int entry(int tid, int q) {
    const int i = tid + q * BLOCK;
    return SIZE % BLOCK == 0 ? i : (WRAP ? i % SIZE : min(i, SIZE - 1));
  }
  template <int SIZE>   // and whether the thread writes one there
  __device__ static __forceinline__ bool writes(int tid, int q) {
    return WRAP || SIZE % BLOCK == 0 || tid + q * BLOCK < SIZE;
  }

  template <class Args>
  __device__ __forceinline__ void begin(const Args& args, int field0, int tid) {
#pragma unroll
    for (int q = 0; q < TT; ++q) {
      const int i = entry<N>(tid, q);
      tw[q] = args.tw[i];
      if constexpr (FUSE) tw2[q] = args.tw2[i];
    }
#pragma unroll
    for (int q = 0; q < TP; ++q) {
      const int k = entry<NF * N>(tid, q);
      const int i = (field0 + k / N) * args.field_stride + args.axis_off + k % N;
      prop[q] = args.prop[i];
      if constexpr (FUSE) prop2[q] = args.prop2[i];
    }
  }

  // conj: lay the conjugate propagators down
  __device__ __forceinline__ void end(bool conj, int tid, float2* s_tw, float2* s_prop, float2* s_tw2,
                                      float2* s_prop2) {
#pragma unroll
    for (int q = 0; q < TT; ++q) {
      const int i = entry<N>(tid, q);
      if (writes<N>(tid, q)) {
        s_tw[i] = tw[q];
        if constexpr (FUSE) s_tw2[i] = tw2[q];
      }
    }
#pragma unroll
    for (int q = 0; q < TP; ++q) {
      const int i = entry<NF * N>(tid, q);
      if (conj) prop[q].y = -prop[q].y;
      if (writes<NF * N>(tid, q)) {
        s_prop[i] = prop[q];
        if constexpr (FUSE) s_prop2[i] = prop2[q];
      }
    }
  }
};

// RK4 coefficients of a half-step: the same for every thread, read before
// any store and kept in scalar registers.
template <int NF>
__device__ __forceinline__ void load_coefficients(const float2* nl, float2 (&co)[NF][kNlCoef]) {
#pragma unroll
  for (int j = 0; j < NF; ++j)
#pragma unroll
    for (int c = 0; c < kNlCoef; ++c) co[j][c] = wave_uniform(nl[j * kNlCoef + c]);
}

// The next step's DftConsts, read behind the pass's first barrier, where a
// batch's descriptor is no longer known to be the same in every lane and 16
// vector registers would hold them through the transforms.  SCALAR (three
// fields of a batch where the registers are short: 16 values a lane, or 192 and
// two half-steps): moved into scalar registers, else those pairs keep 2-39
// values of a lane in scratch memory (now 6 at most; 64 x 256 x 256, literal:
// 3254 -> 3207 us a run).  Elsewhere there is room and the wait for them costs
// 1-2 % (192 x 64 x 64, merged: 2100 / 2123 us).
template <bool SCALAR>
__device__ __forceinline__ DftConsts next_consts(const DftConsts* p) {
  if constexpr (!SCALAR) return *p;
  union {
    float2 w[sizeof(DftConsts) / sizeof(float2)];
    DftConsts k;
  } u;
#pragma unroll
  for (unsigned i = 0; i < sizeof(u.w) / sizeof(float2); ++i)
    u.w[i] = wave_uniform(reinterpret_cast<const float2*>(p)[i]);
  return u.k;
}

// Whether a lane's twiddles stay in registers: where its values leave room.
template <int N1, int NF, int BLOCK>
constexpr bool twiddle_registers() {
  return BLOCK > kBlock ? N1 <= 16 : N1 * NF <= 72;   // (short blocks as kBlock)
}

// Block -> tile map of the x and y passes (slab_tiles says when): blocks go to
// the eight XCDs in turn, and each XCD is given an eighth of the tiles in a
// row, a slab of tau planes.  An x pass and the y pass before or after it then
// work on the same slab in the same XCD, whose L2 still holds part of it.
// (tau lines cross every slab.)  nt, which decides nothing here, is looked at
// beside the flag, which lies in another line of the launch's arguments: both
// lines are then asked for at once (one after the other cost a pass of few
// waves 0.3 us).
template <class Args>
__device__ __forceinline__ unsigned slab_tile(const Args& args, unsigned bx) {
  if (args.nt < 8 || !args.slab) return bx;
  const unsigned per_xcd = gridDim.x / 8u;
  return bx < 8u * per_xcd ? bx % 8u * per_xcd + bx / 8u : bx;   // (the last few tiles as they come)
}

// bx: tile index along the launch's x dimension; field0: first field
// handled (y pass: the block's field); next: a fused pass also applies the
// next step's transform (false: the problem's last step, which ends on its
// own second half-step).  BATCH: args is a descriptor in memory.
template <int N1, int N2, int AX, int NF, int NL, int BLOCK = kBlock, bool BATCH = false>
__device__ __forceinline__ void axis_pass_body(const PassArgs& args, unsigned bx, int field0,
                                               bool next = true) {
  using G = LineGeom<N1, N2, BLOCK>;
  constexpr int N = G::N;
  constexpr int NLM = NL & 3;                  // where the RK4 half-step goes
  constexpr bool MAP = (NL & NL_MAP) != 0;     // transverse mismatch map
  constexpr bool NT = (AX == AX_X) ? bool(BRAHMS_NT_X) : bool(BRAHMS_NT_YT);
  constexpr bool LONG = long_tau_kind(AX);
  constexpr bool FUSE = (NL & NL_FUSE) != 0;   // and the next step's transform
  constexpr bool REG = twiddle_registers<N1, NF, BLOCK>();
  // x lines: a line's N2 lanes are consecutive threads, within one wavefront
  constexpr bool WL = AX == AX_X && N2 <= 64 && 64 % N2 == 0;
  static_assert(NLM != NL_BOTH, "one line: axis_pass_split");
  static_assert(!(MAP && AX == AX_Y), "the transverse map runs only on x or tau");
  constexpr bool LIT = (NL & NL_LIT) != 0;     // two half-steps between the transforms
  static_assert(!FUSE || (NLM == NL_AFTER && !(MAP && !LIT) && !LONG),
                "a fused step pair ends one step and begins the next on one short axis");
  __shared__ float2 lds[G::LDS_ELEMS];
  __shared__ float2 s_tw[N];
  __shared__ float2 s_prop[LONG ? 1 : NF * N];
  __shared__ float2 s_tw2[FUSE ? N : 1];
  __shared__ float2 s_prop2[FUSE ? NF * N : 1];
  // long tau axis: the nt-point twiddles (a and b passes) or the tau
  // propagator (transform pass); the N entries of the block's value of the
  // other index where it has one (ONE), else those of the whole axis
  constexpr bool ONE = (NL & NL_ONE) != 0;
  __shared__ float2 s_long[LONG ? (ONE ? N : kMaxLongT) : 1];

  const int tid = threadIdx.x;
  float2 co[NF][kNlCoef];
  if constexpr (NLM != NL_NONE) load_coefficients<NF>((NLM & NL_BEFORE) != 0 ? args.nl : args.nl2, co);

  const int t = AX == AX_X ? tid % N2 : tid / G::LPB;
  const int li = AX == AX_X ? tid / N2 : tid % G::LPB;
  // tau pass: tiles of consecutive (x, y) columns; concurrently running
  // blocks are spread over the whole plane so that their strided rows fall
  // into many memory channels rather than one narrow address window
  if constexpr (AX == AX_T) bx = unsigned((unsigned long long)bx * args.tile_mul % args.tiles);
  if constexpr (AX == AX_X || AX == AX_Y) bx = slab_tile(args, bx);
  const LineAddr la = line_addr<AX, N>(args, bx * unsigned(G::LPB) + unsigned(li));
  const bool valid = la.valid;
  const unsigned lidx = la.lidx;
  const float2* fin[NF];
  float2* fout[NF];
#pragma unroll
  for (int j = 0; j < NF; ++j) {
    fin[j] = args.f[field0 + j];
    fout[j] = args.fo[field0 + j];
  }
  const unsigned idx0 = la.base + unsigned(t) * la.estride;
  const unsigned estep = unsigned(N2) * la.estride;
  // transverse-map offset of slot 0 (x pass: slot e adds N2 e entries; tau
  // pass: the same column for every slot, its three factors are read once)
  constexpr bool COLUMN = AX == AX_T || LONG;
  const unsigned plane = unsigned(args.nx) * unsigned(args.ny);
  const unsigned map_bytes = MAP ? (idx0 % plane) * 8u : 0u;
  // a line's LDS row (lines of one lane exchange nothing: no row)
  float2* lbuf = (N2 > 1) ? lds + li * G::LSTRIDE : lds;
  const DftConsts K = *args.consts;

  const unsigned field_bytes = unsigned(args.nx) * unsigned(args.ny) * unsigned(args.nt) * 8u;
  const unsigned lane_bytes = idx0 * 8u;
  const unsigned slot_bytes = estep * 8u;
  __amdgpu_buffer_rsrc_t rin[NF], rout[NF];
#pragma unroll
  for (int j = 0; j < NF; ++j) {
    rin[j] = field_rsrc(fin[j], field_bytes);
    rout[j] = field_rsrc(fout[j], field_bytes);
  }
  float2 v[NF][N1];
  auto load_fields = [&]() {
#pragma unroll
    for (int j = 0; j < NF; ++j) {
#pragma unroll
      for (int e = 0; e < N1; ++e) v[j][e] = load_slot<NT>(rin[j], lane_bytes, unsigned(e) * slot_bytes);
    }
  };
  if constexpr (LONG) {
    // args.tw is the nt-point row exp(-2 pi i m / nt); the line transforms
    // of length N take every (nt / N)-th entry
    static_assert(N <= BLOCK, "one twiddle per thread");
    const int nt = args.nt;
    const float2* whole = AX == AX_TB ? args.prop + field0 * args.field_stride + args.axis_off : args.tw;
    const float2 w_tw = args.tw[min(tid, N - 1) * (nt / N)];
    if constexpr (ONE) {
      // entry k of the block: a k_b (b passes) or k_b + B k_a (a pass)
      const unsigned k = unsigned(min(tid, N - 1));
      float2 w = whole[AX == AX_TB ? lidx + unsigned(nt / N) * k : (lidx * k) & unsigned(nt - 1)];
      load_fields();
      if (AX == AX_TB && args.conj) w.y = -w.y;
      if (tid < N) {
        s_tw[tid] = w_tw;
        s_long[tid] = w;
      }
    } else {
      constexpr int U = 2;   // (nt is a multiple of 2 BLOCK)
      float2 w_long[U];
#pragma unroll
      for (int q = 0; q < U; ++q) w_long[q] = whole[tid + q * BLOCK];
      load_fields();
      if (tid < N) s_tw[tid] = w_tw;
      for (int i = tid;; i += U * BLOCK) {
#pragma unroll
        for (int q = 0; q < U; ++q) {
          if (AX == AX_TB && args.conj) w_long[q].y = -w_long[q].y;
          s_long[i + q * BLOCK] = w_long[q];
        }
        if (i + U * BLOCK >= nt) break;
#pragma unroll
        for (int q = 0; q < U; ++q) w_long[q] = whole[i + (U + q) * BLOCK];
      }
    }
  } else {
    StageTables<N, NF, BLOCK, FUSE, NF == 1 && !BATCH && BLOCK == kBlock> st;
    st.begin(args, field0, tid);
    load_fields();
    st.end(args.conj != 0, tid, s_tw, s_prop, s_tw2, s_prop2);
  }
  __syncthreads();  // s_tw, s_prop staged
  LaneTwiddles<N1, N2, REG> tw;
  tw.init(s_tw, t);

  if constexpr ((NLM & NL_BEFORE) != 0) {
    __amdgpu_buffer_rsrc_t rmap;
    float2 w[3];
    if constexpr (MAP) {
      rmap = field_rsrc(args.map, 3u * plane * 8u);
      if constexpr (COLUMN) map_factors(rmap, plane, map_bytes, 0u, w);
    }
#pragma unroll
    for (int e = 0; e < N1; ++e) {
      float2 y[NF];
#pragma unroll
      for (int j = 0; j < NF; ++j) y[j] = v[j][e];
      if (e > 0) point_link<NF>(y, v, e - 1);
      if constexpr (MAP) {
        if constexpr (!COLUMN) map_factors(rmap, plane, map_bytes, unsigned(N2 * e) * 8u, w);
        rk4_point<NF, true>(y, co, w);
      } else {
        rk4_point<NF>(y, co);
      }
#pragma unroll
      for (int j = 0; j < NF; ++j) v[j][e] = y[j];
    }
  }

  if constexpr (LONG) {
    const unsigned nb = unsigned(args.nt) / unsigned(N);
    auto factor = [&](int k) {   // of element k of the line
      if constexpr (ONE) return s_long[k];
      else if constexpr (AX == AX_TB) return s_long[lidx + nb * unsigned(k)];
      else return s_long[(lidx * unsigned(k)) & unsigned(args.nt - 1)];
    };
#pragma unroll
    for (int j = 0; j < NF; ++j) {
      if constexpr (AX == AX_TAF) {
        // B-point transform, then exp(-2 pi i a k_b / nt) on output k_b
        line_fft<N1, N2, false, WL>(v[j], tw, t, lbuf, K);
#pragma unroll
        for (int e = 0; e < N1; ++e)
          v[j][e] = cmul(v[j][e], factor(t + N2 * e));
      } else if constexpr (AX == AX_TAI) {
        // conjugate twiddle, then the inverse B-point transform
#pragma unroll
        for (int e = 0; e < N1; ++e)
          v[j][e] = cmulc(v[j][e], factor(t + N2 * e));
        line_fft<N1, N2, true, WL>(v[j], tw, t, lbuf, K);
      } else {
        // A-point transform over a gives frequency k = k_b + B k_a in slot k_a
        line_fft<N1, N2, false, WL>(v[j], tw, t, lbuf, K);
#pragma unroll
        for (int e = 0; e < N1; ++e) v[j][e] = cmul(v[j][e], factor(t + N2 * e));
        line_fft<N1, N2, true, WL>(v[j], tw, t, lbuf, K);
      }
    }
  } else {
    line_trip<N1, N2, NF, WL, false>(v, tw, t, lbuf, s_prop, K);
  }

  if constexpr ((NLM & NL_AFTER) != 0) {
    // with a map, lines past the last one are done (nothing after this waits
    // for them): were they to go on to the stores, the compiler would move the
    // points' arithmetic down to the valid lines' stores, away from its factors
    if (MAP && !FUSE && !valid) return;
    // (only unfused steps are asked for their values before the half-step)
    if (!FUSE && args.pre[0] != nullptr && valid) {
#pragma unroll
      for (int j = 0; j < NF; ++j) {
        const __amdgpu_buffer_rsrc_t rp = field_rsrc(args.pre[j], field_bytes);
#pragma unroll
        for (int e = 0; e < N1; ++e) store_slot<NT>(rp, lane_bytes, unsigned(e) * slot_bytes, v[j][e]);
      }
    }
    auto half_step = [&](const float2* map) {
    __amdgpu_buffer_rsrc_t rmap;
    float2 w[3];
    if constexpr (MAP) {
      rmap = field_rsrc(map, 3u * plane * 8u);
      if constexpr (COLUMN) map_factors(rmap, plane, map_bytes, 0u, w);
    }
#pragma unroll
    for (int e = 0; e < N1; ++e) {
      float2 y[NF];
#pragma unroll
      for (int j = 0; j < NF; ++j) y[j] = v[j][e];
      // (after the transforms a schedule barrier between points keeps
      // fewer registers live than the link above, where exchanges follow that
      // hold the points' arithmetic in place)
      if constexpr (FUSE && N2 == 1) {
        if (e > 0) point_link<NF>(y, v, e - 1);
      } else {
        __builtin_amdgcn_sched_barrier(0);
      }
      if constexpr (MAP) {
        if constexpr (!COLUMN) map_factors(rmap, plane, map_bytes, unsigned(N2 * e) * 8u, w);
        rk4_point<NF, true>(y, co, w);
      } else {
        rk4_point<NF>(y, co);
      }
#pragma unroll
      for (int j = 0; j < NF; ++j) v[j][e] = y[j];
    }
    };
    half_step(args.map);
    if constexpr (FUSE) if (next) {
      if constexpr (LIT) {
        load_coefficients<NF>(args.nl, co);
        half_step(args.map2);
      }
      // the next step's first transform along this axis
      __builtin_amdgcn_sched_barrier(0);
      const DftConsts K2 =
          next_consts<BATCH && NF == 3 && (N1 == 16 || (N1 * N2 == 192 && LIT))>(args.consts2);
      LaneTwiddles<N1, N2, REG> tw2;
      tw2.init(s_tw2, t);
      line_trip<N1, N2, NF, WL, false>(v, tw2, t, lbuf, s_prop2, K2);
    }
  }
  if (valid) {
#pragma unroll
    for (int j = 0; j < NF; ++j)
#pragma unroll
      for (int e = 0; e < N1; ++e) store_slot<NT>(rout[j], lane_bytes, unsigned(e) * slot_bytes, v[j][e]);
  }
}

// ---------------------------------------------------------------------------
// The pass with one field per thread: NF groups of T threads, group f with
// field f's values of the block's T / N2 lines, each group transforming its
// field; for the RK4 step the groups lay their values down in LDS, every
// thread takes the points e = f, f + NF, ... of its place in the line with
// all their fields, and lays the results back.  The arithmetic of every value
// is that of axis_pass_body, so the two give the same bits and a launch may
// take either.  It is for launches that leave SIMDs with less than two waves
// (narrow_launch): their time is the serial chain of one wave, and here a
// wave's chain is 1 / NF as long and there are NF times as many waves.
// ---------------------------------------------------------------------------
template <int N1, int N2, int AX, int NF, int NL, int T>
__device__ __forceinline__ void axis_pass_split_body(const PassArgs& args, unsigned bx, bool next = true) {
  using G = LineGeom<N1, N2, T>;
  constexpr int N = G::N, BLOCK = NF * T;
  constexpr int NLM = NL & 3;
  constexpr bool MAP = (NL & NL_MAP) != 0;
  constexpr bool NT = (AX == AX_X) ? bool(BRAHMS_NT_X) : bool(BRAHMS_NT_YT);
  constexpr bool FUSE = (NL & NL_FUSE) != 0;
  constexpr bool WL = AX == AX_X && T == 64 && N2 <= 64 && 64 % N2 == 0;
  static_assert(NLM != NL_NONE && !long_tau_kind(AX) && T % 64 == 0, "a pass with an RK4 step on one line axis");
  constexpr bool LIT = (NL & NL_LIT) != 0;
  static_assert(!(MAP && (NLM == NL_BOTH || AX == AX_Y)),
                "the transverse map runs only with a half-step per pass on x or tau");
  // a group's LDS: its lines' exchange rows, or its values around the RK4 step
  constexpr int XS = N2 > 1 ? G::LDS_ELEMS : N1 * T;
  static_assert(XS >= N1 * T, "the exchange rows hold the group's values");
  __shared__ float2 lds[NF * XS];
  __shared__ float2 s_tw[N], s_prop[NF * N], s_tw2[FUSE ? N : 1], s_prop2[FUSE ? NF * N : 1];

  const int tid = threadIdx.x;
  const int f = __builtin_amdgcn_readfirstlane(tid / T);   // (T is a multiple of the wave)
  const int g = tid % T;
  float2 co[NF][kNlCoef];
  load_coefficients<NF>((NLM & NL_BEFORE) != 0 ? args.nl : args.nl2, co);
  const int t = AX == AX_X ? g % N2 : g / G::LPB;
  const int li = AX == AX_X ? g / N2 : g % G::LPB;
  if constexpr (AX != AX_T) bx = slab_tile(args, bx);
  const LineAddr la = line_addr<AX, N>(args, bx * unsigned(G::LPB) + unsigned(li));
  const unsigned idx0 = la.base + unsigned(t) * la.estride;
  const unsigned estep = unsigned(N2) * la.estride;
  const unsigned field_bytes = unsigned(args.nx) * unsigned(args.ny) * unsigned(args.nt) * 8u;
  const unsigned lane_bytes = idx0 * 8u, slot_bytes = estep * 8u;
  const __amdgpu_buffer_rsrc_t rin = field_rsrc(args.f[f], field_bytes), rout = field_rsrc(args.fo[f], field_bytes);
  const DftConsts K = *args.consts;
  float2* mine = lds + f * XS;
  float2* lbuf = (N2 > 1) ? mine + li * G::LSTRIDE : mine;

  float2 v[N1];
  {
    StageTables<N, NF, BLOCK, FUSE> st;
    st.begin(args, 0, tid);
#pragma unroll
    for (int e = 0; e < N1; ++e) v[e] = load_slot<NT>(rin, lane_bytes, unsigned(e) * slot_bytes);
    st.end(false, tid, s_tw, s_prop, s_tw2, s_prop2);
  }
  // transverse phase factors of this thread's points
  constexpr int P = (N1 + NF - 1) / NF;
  float2 wm[MAP ? P : 1][3], wm2[MAP && LIT ? P : 1][3];
  if constexpr (MAP) {
    const unsigned plane = unsigned(args.nx) * unsigned(args.ny);
    const unsigned xy0 = idx0 % plane;
#pragma unroll
    for (int k = 0; k < P; ++k) {
      const unsigned xy = xy0 + (AX == AX_T ? 0u : unsigned(N2 * min(f + NF * k, N1 - 1)));
#pragma unroll
      for (int s = 0; s < 3; ++s) {
        wm[k][s] = (AX == AX_T && k > 0) ? wm[0][s] : args.map[s * plane + xy];
        if constexpr (LIT) wm2[k][s] = (AX == AX_T && k > 0) ? wm2[0][s] : args.map2[s * plane + xy];
      }
    }
  }
  __syncthreads();  // s_tw, s_prop staged
  LaneTwiddles<N1, N2, true> tw;
  tw.init(s_tw, t);

  // (two: NL_LIT, the next step's first half-step follows on the same points)
  auto rk4 = [&](bool two) {
    line_sync<WL>();   // this group's exchange rows are free
#pragma unroll
    for (int e = 0; e < N1; ++e) mine[e * T + g] = v[e];
    __syncthreads();
    float2 y[P][NF];
#pragma unroll
    for (int k = 0; k < P; ++k) {
      const int e = f + NF * k;
      if (N1 % NF == 0 || e < N1) {
#pragma unroll
        for (int j = 0; j < NF; ++j) y[k][j] = lds[j * XS + e * T + g];
        if constexpr (MAP) rk4_point<NF, true>(y[k], co, wm[k]);
        else rk4_point<NF>(y[k], co);
        if constexpr (!LIT) {
#pragma unroll
          for (int j = 0; j < NF; ++j) lds[j * XS + e * T + g] = y[k][j];
        }
      }
    }
    if constexpr (LIT) {
      if (two) load_coefficients<NF>(args.nl, co);
#pragma unroll
      for (int k = 0; k < P; ++k) {
        const int e = f + NF * k;
        if (N1 % NF == 0 || e < N1) {
          if (two) {
            if constexpr (MAP) rk4_point<NF, true>(y[k], co, wm2[k]);
            else rk4_point<NF>(y[k], co);
          }
#pragma unroll
          for (int j = 0; j < NF; ++j) lds[j * XS + e * T + g] = y[k][j];
        }
      }
    }
    __syncthreads();
#pragma unroll
    for (int e = 0; e < N1; ++e) v[e] = mine[e * T + g];
  };
  float2 (&v1)[1][N1] = reinterpret_cast<float2 (&)[1][N1]>(v);

  if constexpr ((NLM & NL_BEFORE) != 0) rk4(false);
  line_trip<N1, N2, 1, WL, false>(v1, tw, t, lbuf, s_prop + f * N, K);
  if constexpr ((NLM & NL_AFTER) != 0) {
    if constexpr (NLM == NL_BOTH) load_coefficients<NF>(args.nl2, co);
    if (!FUSE && args.pre[0] != nullptr && la.valid) {
      const __amdgpu_buffer_rsrc_t rp = field_rsrc(args.pre[f], field_bytes);
#pragma unroll
      for (int e = 0; e < N1; ++e) store_slot<NT>(rp, lane_bytes, unsigned(e) * slot_bytes, v[e]);
    }
    rk4(next);
    if constexpr (FUSE) if (next) {
      const DftConsts K2 = *args.consts2;
      tw.init(s_tw2, t);
      line_trip<N1, N2, 1, WL, false>(v1, tw, t, lbuf, s_prop2 + f * N, K2);
    }
  }
  if (la.valid) {
#pragma unroll
    for (int e = 0; e < N1; ++e) store_slot<NT>(rout, lane_bytes, unsigned(e) * slot_bytes, v[e]);
  }
}

// Threads per field group of the split pass: one wave on x (its lines are
// contiguous and exchange within the wave); on y and tau as many as give row
// segments of 16 lines (128 B): 64^3 points and two fields, tau: 6.1 us with
// 16 lines, 7.8 us with 8.
__host__ __device__ constexpr int split_threads(int n2, int ax) {
  return ax == AX_X || 16 * n2 < 64 ? 64 : (16 * n2 > 256 ? 256 : 16 * n2);
}

// Whether a pass over `lines` lines of n2 lanes takes one field per thread:
// when the fields-together pass would have less than two waves for each of
// the 1024 SIMDs.  Below that a SIMD's time is the chain of its one wave
// (which issues at most every other slot), and splitting it wins: 32^3 and
// two fields, fused x pass: 64 waves, 4.6 against 7.3 us; 64^3: 512 waves,
// 5.6 / 7.8; 128 x 128 x 64: 1024 waves, 13.1 / 17.3; at 2048 waves the two
// are even (same grid, tau: 11.5 / 11.4; 128^3 and three fields, x: 32.8 /
// 29.8) and beyond it the fields-together pass wins, having no exchange of
// values around the RK4 step (256^3, x: 225 / 180).
__host__ __device__ constexpr bool narrow_launch(long long lines, int n2) {
  return lines * n2 < 2LL * 1024 * 64;
}

// Whether a split has passes with the fields together at all: not with 36
// values per lane (lengths 72 and 144), where three fields take 394 registers
// and one block fills a CU; one field per thread is as fast or faster at any
// size (144 x 192 x 192 and three fields, x: 229 -> 114 us; 192 x 192 x 144
// and two, tau: 109 -> 64; 72 x 256 x 256, x: 149 / 148; 256 x 256 x 72 and
// three, tau: 137 / 142).
template <int N1>
constexpr bool together_split() {
  return N1 <= 24;
}

// Threads per block of the wide linear passes (schedule field `wide`): twice
// the lines of a kBlock block, so y and tau rows are read in segments twice
// as long; their LDS allows two blocks per CU.
constexpr int kWideBlock = 2 * kBlock;

__host__ __device__ inline int table_row_stride(int nf, int nx, int ny, int nt) {
  return (nf + 1) * (nx + ny + nt) + int(sizeof(DftConsts) / sizeof(float2));
}

// Blocks per CU a pass kernel of N1 values per lane and BLOCK threads is
// compiled for (the second argument of its launch bounds).
template <int N1, int N2, int BLOCK>
constexpr int pass_min_blocks() {
  return BLOCK > kBlock ? 2 : (N1 > 24 ? 1 : (N1 >= 18 ? 2 : BRAHMS_MIN_BLOCKS));
}

// Whether the wide linear passes of a split fit the LDS of one CU (160 KB):
// not for 36 values per lane, whose rows of 512 lanes would take 185-223 KB.
// Such axes run their linear passes with kBlock threads whatever the
// schedule's `wide` bit says (the results are the same either way).
template <int N1>
constexpr bool wide_split() {
  return N1 <= 24;
}

// One pass of one problem; BLOCK threads per block (kBlock, or kWideBlock
// for the wide linear passes of the schedule field `wide`).
template <int N1, int N2, int AX, int NF, int NL, int BLOCK = kBlock>
__global__ __launch_bounds__(BLOCK, (pass_min_blocks<N1, N2, BLOCK>())) void axis_pass(PassArgs args) {
  // passes with one field per block take it from blockIdx.z
  constexpr bool per_field = NF == 1;
  axis_pass_body<N1, N2, AX, NF, NL, BLOCK>(args, blockIdx.x, per_field ? int(blockIdx.z) : 0);
}

// One pass over a group of problems of the same shape (a batch): descs[i]
// describes problem i at this step; passes over all fields take the problem
// from blockIdx.y, passes with one field per block from blockIdx.z / nf.  Problems whose own step count
// is reached (step >= nz) leave at once.
template <int N1, int N2, int AX, int NF, int NL, int BLOCK = kBlock>
__global__ __launch_bounds__(BLOCK, (pass_min_blocks<N1, N2, BLOCK>())) void axis_pass_batched(
    const PassArgs* descs, long long step, int nf) {
  // linear y and long-tau passes take one field per block: problem and field
  // from blockIdx.z
  constexpr bool per_field = NF == 1;
  const unsigned inst = per_field ? blockIdx.z / unsigned(nf) : blockIdx.y;
  const PassArgs& a = descs[inst];
  if (step >= a.nz) return;
  // a fused pass ends the problem's last step without the next transform
  axis_pass_body<N1, N2, AX, NF, NL, BLOCK, true>(a, blockIdx.x, per_field ? int(blockIdx.z % unsigned(nf)) : 0,
                                                  step + 1 < a.nz);
}

// The passes with one field per thread, of one problem and of a group.
template <int N1, int N2, int AX, int NF, int NL>
__global__ __launch_bounds__((NF * split_threads(N2, AX))) void axis_pass_split(PassArgs args) {
  axis_pass_split_body<N1, N2, AX, NF, NL, split_threads(N2, AX)>(args, blockIdx.x);
}

template <int N1, int N2, int AX, int NF, int NL>
__global__ __launch_bounds__((NF * split_threads(N2, AX))) void axis_pass_split_batched(
    const PassArgs* descs, long long step, int nf) {
  const PassArgs& a = descs[blockIdx.y];
  if (step >= a.nz) return;
  axis_pass_split_body<N1, N2, AX, NF, NL, split_threads(N2, AX)>(a, blockIdx.x, step + 1 < a.nz);
}

// ---------------------------------------------------------------------------
// Plane waves (nx = ny = 1): the field is one tau line, nothing else depends
// on it, and a block keeps it in registers over `count` steps: half-step, FFT
// . P . IFFT, half-step, with the tables of consecutive rows (args: the first
// one's).  merged: a step's first half-step is part of the previous one's
// second; `first` says whether the first step here has its own.  One wave per
// field transforms (its lanes past the line repeat it), and the RK4 points
// are spread over all the block's threads; a step's time is this serial chain
// (no memory traffic to speak of), with the next step's tables loaded beside
// it.  nt = 256, two fields, literal half-steps: 19.5 us a step as a launch
// per step of one wave of 32 values a lane, 10.5 us as a launch per step with
// one field per wave, 4.0 us here.
// ---------------------------------------------------------------------------
template <int N1, int N2, int NF>
__device__ __forceinline__ void line_steps_body(const PassArgs& args, int count, bool merged, bool first) {
  constexpr int T = 64, BLOCK = NF * T;
  using G = LineGeom<N1, N2, T>;
  constexpr int N = G::N;
  static_assert(N2 <= T, "a line within one wave");
  __shared__ float2 lds[NF * (N2 > 1 ? G::LDS_ELEMS : 1)];
  __shared__ float2 s_val[NF][N];
  __shared__ float2 s_tw[N], s_prop[NF * N];
  const int tid = threadIdx.x;
  const int f = __builtin_amdgcn_readfirstlane(tid / T);
  const int t = tid % N2, li = tid % T / N2;
  const int row = table_row_stride(NF, 1, 1, N);
  float2* lbuf = (N2 > 1) ? lds + f * G::LDS_ELEMS + li * G::LSTRIDE : lds;
  const __amdgpu_buffer_rsrc_t r = field_rsrc(args.f[f], unsigned(N) * 8u);
  const unsigned lane_bytes = unsigned(t) * 8u;
  PassArgs a = args;   // (advanced row by row)
  StageTables<N, NF, BLOCK, false> st;
  st.begin(a, 0, tid);
  float2 v[1][N1];
#pragma unroll
  for (int e = 0; e < N1; ++e) v[0][e] = load_slot<false>(r, lane_bytes, unsigned(N2 * e) * 8u);
  LaneTwiddles<N1, N2, true> tw;

  auto rk4 = [&](const float2* nl) {
    float2 co[NF][kNlCoef];
    load_coefficients<NF>(nl, co);
    if (li == 0) {
#pragma unroll
      for (int e = 0; e < N1; ++e) s_val[f][t + N2 * e] = v[0][e];
    }
    __syncthreads();
    for (int q = tid; q < N; q += BLOCK) {
      float2 y[NF];
#pragma unroll
      for (int j = 0; j < NF; ++j) y[j] = s_val[j][q];
      rk4_point<NF>(y, co);
#pragma unroll
      for (int j = 0; j < NF; ++j) s_val[j][q] = y[j];
    }
    __syncthreads();
#pragma unroll
    for (int e = 0; e < N1; ++e) v[0][e] = s_val[f][t + N2 * e];
  };
  for (int s = 0; s < count; ++s) {
    __syncthreads();   // the previous step's tables and values are read
    st.end(false, tid, s_tw, s_prop, s_tw, s_prop);
    const DftConsts K = *a.consts;
    const float2 *nl = a.nl, *nl2 = a.nl2;
    a.tw += row;
    a.prop += row;
    a.consts = reinterpret_cast<const DftConsts*>(reinterpret_cast<const float2*>(a.consts) + row);
    a.nl += 2 * NF * kNlCoef;
    a.nl2 += 2 * NF * kNlCoef;
    if (s + 1 < count) st.begin(a, 0, tid);
    if (!merged || (s == 0 && first)) rk4(nl);   // (its barriers stand behind the tables')
    else __syncthreads();
    tw.init(s_tw, t);
    line_trip<N1, N2, 1, true, false>(v, tw, t, lbuf, s_prop + f * N, K);
    rk4(nl2);
  }
  if (li == 0) {
    const __amdgpu_buffer_rsrc_t ro = field_rsrc(args.fo[f], unsigned(N) * 8u);
#pragma unroll
    for (int e = 0; e < N1; ++e) store_slot<false>(ro, lane_bytes, unsigned(N2 * e) * 8u, v[0][e]);
  }
}

template <int N1, int N2, int NF>
__global__ __launch_bounds__(NF * 64) void line_steps(PassArgs args, int count, int merged, int first) {
  line_steps_body<N1, N2, NF>(args, count, merged != 0, first != 0);
}

// Steps step .. step + count - 1 of a group (descs: of the first step).
template <int N1, int N2, int NF>
__global__ __launch_bounds__(NF * 64) void line_steps_batched(const PassArgs* descs, long long step, int count,
                                                              int merged) {
  const PassArgs& a = descs[blockIdx.x];
  const long long left = a.nz - step;
  if (left <= 0) return;
  line_steps_body<N1, N2, NF>(a, int(min((long long)count, left)), merged != 0, step == 0);
}

// ---------------------------------------------------------------------------
// Per-step tables, formed in double precision.
//
// Propagator of field j along one axis for step n (z_n = n dz):
//   P_n(k) = s * U(z_{n+1}, k) * conj(U(z_n, k)),   U(z, k) = fl32(exp(i phi(k) z))
// with phi the imaginary part of that axis's share of the symbol Lambda_j,
// the phase reduced to a turn in double before the sine and cosine, and s the
// 1/N normalisation (times exp(-alpha dz/2) on the tau axis).  Because U is
// rounded at every z_n separately, the phase rounding errors of consecutive
// steps cancel (a telescoping product) instead of accumulating coherently.
//
// The propagator entries themselves, the transform twiddles, the register-DFT
// constants and the RK4 coefficients (see rk4_point; Phi(z) = Phi_n +
// dk_n (z - z_n) is the integrated mismatch) are rounded to float
// stochastically, with a
// counter-based hash of (step, entry) as the random source, so that their
// rounding errors are independent from one z-step to the next; a fixed
// rounding would repeat the same error every step and add up linearly.
//
// Row layout of one step (float2 units): [nf][nx | ny | nt] propagators,
// [nx | ny | nt] twiddles, 8 float2 of DftConsts.
// ---------------------------------------------------------------------------
struct FieldCoef {
  double kappa, diffraction, tan_rho, delay, k2, k3, alpha;
};

struct TableArgs {
  float2* rows;          // [count][row_stride]
  float2* nl;            // [count][2][nf][6]
  const double* phi0;    // Phi_n prefix (profile) or null
  const double* dk;      // dk_n (profile) or null
  long n0;               // first step of the rows (unless n0_dev is set)
  const long long* n0_dev;  // device copies of n0 and merge_last (graph
                            // replays), or null
  long long merge_last;  // steps n < merge_last get the merged second
                         // half-step coefficients; -1: none (constant dk only)
  int count;
  int nx, ny, nt, nf;
  int row_stride;
  double dz, dx, dy, dt, dk_const;
  FieldCoef fc[3];
};

__device__ inline long table_n0(const TableArgs& a) {
  return a.n0_dev != nullptr ? long(a.n0_dev[0]) : a.n0;
}

__device__ inline long long table_merge_last(const TableArgs& a) {
  return a.n0_dev != nullptr ? a.n0_dev[1] : a.merge_last;
}

// sin and cos of a phase of any size: its part of a turn, a / (2 pi) minus the
// nearest integer, in two-term arithmetic (the product's rounding error and
// the rest of 1 / (2 pi) are added back after the integer is gone), then
// sincospi.  (With fmod and sincos the table kernel of one step of 32^3 took
// 8.2 us, most of a call's time; it is a chain of FP64 instructions.)
__device__ inline void phase_sincos(double a, double* sn, double* cs) {
  const double inv = 0.15915494309189534561, inv_lo = -9.8393381170937e-18;
  const double t = a * inv;
  const double lo = fma(a, inv_lo, fma(a, inv, -t));
  const double r = (t - rint(t)) + lo;
  sincospi(2.0 * r, sn, cs);
}

__device__ inline double ang_freq(int m, int n, double d) {
  const int mm = (m >= (n + 1) / 2) ? m - n : m;
  return 6.283185307179586476925286766559 * double(mm) / (double(n) * d);
}

__device__ inline double2 rounded_unit(double theta) {
  double s, c;
  phase_sincos(theta, &s, &c);
  return make_double2(double(float(c)), double(float(s)));
}

// 32-bit integer hash (xorshift-multiply finaliser).
__device__ inline unsigned mix32(unsigned x) {
  x ^= x >> 16;
  x *= 0x7feb352du;
  x ^= x >> 15;
  x *= 0x846ca68bu;
  x ^= x >> 16;
  return x;
}

__device__ inline unsigned entry_bits(long n, unsigned slot) {
  return mix32(mix32(unsigned(n) * 0x9e3779b1u ^ unsigned(n >> 32)) ^ (slot * 0x85ebca6bu + 0x632be5abu));
}

// Round v to one of its two float neighbours, up with probability equal to
// the distance from the lower one (unbiased), using 24 random bits.
__device__ inline float stochastic_round(double v, unsigned bits) {
  const float f = float(v);
  const double d = double(f);
  if (d == v) return f;
  float lo, hi;
  if (d < v) {
    lo = f;
    hi = nextafterf(f, HUGE_VALF);
  } else {
    hi = f;
    lo = nextafterf(f, -HUGE_VALF);
  }
  const double p = (v - double(lo)) / (double(hi) - double(lo));
  const double u = double(bits >> 8) * (1.0 / 16777216.0);
  return (u < p) ? hi : lo;
}

__device__ __forceinline__ void step_tables_body(const TableArgs& a, long gid) {
  const int per_field = a.nx + a.ny + a.nt;
  const int per_step = (a.nf + 1) * per_field + 1;  // + one thread for DftConsts
  const long nrow = long(a.count) * per_step;
  if (gid < nrow) {
    const int s = int(gid / per_step);
    const int r = int(gid % per_step);
    const long n = table_n0(a) + s;
    float2* row = a.rows + long(s) * a.row_stride;
    if (r == per_step - 1) {
      // register-DFT constants of this step
      const double v[6] = {0.70710678118654752440, 0.92387953251128675613, 0.38268343236508977173,
                           0.86602540378443864676, 0.96592582628906828675, 0.25881904510252076235};
      float* out = reinterpret_cast<float*>(row + (a.nf + 1) * per_field);
      for (int k = 0; k < 6; ++k) out[k] = stochastic_round(v[k], entry_bits(n, 0x40000000u + k));
      out[6] = stochastic_round(0.41421356237309504880, entry_bits(n, 0x40000006u));   // tan(pi/8)
      out[7] = 0.f;
      // cos and sin of 10, 20 and 40 degrees (radices with a factor 9)
      const double w[6] = {0.98480775301220805937, 0.17364817766693034885, 0.93969262078590838405,
                           0.34202014332566873304, 0.76604444311897803520, 0.64278760968653932632};
      for (int k = 0; k < 6; ++k) out[8 + k] = stochastic_round(w[k], entry_bits(n, 0x40000008u + k));
      out[14] = 0.f;
      out[15] = 0.f;
      return;
    }
    int m = r % per_field;
    int nax, axis;
    double d;
    if (m < a.nx) {
      axis = 0; nax = a.nx; d = a.dx;
    } else if (m < a.nx + a.ny) {
      axis = 1; nax = a.ny; d = a.dy; m -= a.nx;
    } else {
      axis = 2; nax = a.nt; d = a.dt; m -= a.nx + a.ny;
    }
    if (r >= a.nf * per_field) {
      // forward twiddle exp(-2 pi i m / nax) of this axis
      double sn, cs;
      sincospi(2.0 * double(m) / double(nax), &sn, &cs);
      const unsigned slot = 2u * unsigned(r);
      row[r] = make_float2(stochastic_round(cs, entry_bits(n, slot)),
                           stochastic_round(-sn, entry_bits(n, slot + 1)));
      return;
    }
    const int j = r / per_field;
    const FieldCoef& f = a.fc[j];
    const double k = ang_freq(m, nax, d);
    double phi, scale;
    if (axis == 0) {
      phi = -f.diffraction * k * k - f.tan_rho * k;
      scale = 1.0 / a.nx;
    } else if (axis == 1) {
      phi = -f.diffraction * k * k;
      scale = 1.0 / a.ny;
    } else {
      phi = -f.delay * k + 0.5 * f.k2 * k * k - (f.k3 / 6.0) * k * k * k;
      scale = exp(-0.5 * f.alpha * a.dz) / a.nt;
    }
    const double2 u1 = rounded_unit(phi * (double(n + 1) * a.dz));
    const double2 u0 = rounded_unit(phi * (double(n) * a.dz));
    const double re = (u1.x * u0.x + u1.y * u0.y) * scale;
    const double im = (u1.y * u0.x - u1.x * u0.y) * scale;
    // stochastic, like the other per-step constants: an entry that is the
    // same at every step (zero frequency, where it is the 1/n scale, which is
    // inexact for n = 96) would otherwise be rounded the same way every step
    // and its error would grow linearly with the number of steps
    const unsigned slot = 2u * unsigned(r);
    row[r] = make_float2(stochastic_round(re, entry_bits(n, slot)),
                         stochastic_round(im, entry_bits(n, slot + 1)));
    return;
  }
  const long g2 = gid - nrow;
  // RK4 coefficients: one thread each
  const long nco = long(a.count) * 2 * a.nf * kNlCoef;
  if (g2 >= nco) return;
  const int k = int(g2 % kNlCoef);
  const long g3 = g2 / kNlCoef;
  const int s = int(g3 / (2 * a.nf));
  const int half = int((g3 / a.nf) % 2);
  const int j = int(g3 % a.nf);
  const long n = table_n0(a) + s;
  double phi_n, dkn;
  if (a.dk != nullptr) {
    phi_n = a.phi0[n];
    dkn = a.dk[n];
  } else {
    dkn = a.dk_const;
    phi_n = dkn * (double(n) * a.dz);
  }
  // sigma_j: exp(-i Phi) on the sum-frequency field, exp(+i Phi) on the others
  double sigma;
  if (a.nf == 3) sigma = (j == 0) ? -1.0 : 1.0;
  else sigma = (j == 0) ? 1.0 : -1.0;
  // merged: one step of size dz from z_n + dz/2 (stages at dz/2, dz, 3 dz/2
  // past z_n; only for a constant dk, so Phi stays linear across z_{n+1})
  const bool merged = half == 1 && n < table_merge_last(a);
  const double h = merged ? a.dz : 0.5 * a.dz;
  const double kap = a.fc[j].kappa;
  // weights of a1, a2, a3, b1, b2, b4 and the stage (z_a, z_a + h/2, z_a + h)
  // of each one's c_j
  const double w = k < 2 ? h / 2 : (k == 2 ? h : (k == 4 ? h / 3 : h / 6));
  const int stage = k == 0 || k == 3 ? 0 : (k == 5 ? 2 : 1);
  const double off = merged ? (0.5 + 0.5 * double(stage)) * a.dz                   // z - z_n
                            : (double(half) * 2.0 + double(stage)) * 0.25 * a.dz;
  double sn, cs;
  phase_sincos(phi_n + dkn * off, &sn, &cs);
  // i kappa (cos + i sigma sin) = kappa (-sigma sin + i cos)
  const unsigned slot = 0x50000000u + unsigned((half * a.nf + j) * kNlCoef + k) * 2u;
  a.nl[g2] = make_float2(stochastic_round(w * (-kap * sigma * sn), entry_bits(n, slot)),
                         stochastic_round(w * (kap * cs), entry_bits(n, slot + 1)));
}

// Threads of a table launch over `count` steps.
inline long table_threads(int count, int nf, int per_field) {
  return long(count) * ((nf + 1) * per_field + 1 + 2 * nf * kNlCoef);
}

static __global__ void step_tables(TableArgs a) {
  step_tables_body(a, long(blockIdx.x) * blockDim.x + threadIdx.x);
}

// Tables of several problems: problem blockIdx.y uses targs[blockIdx.y].
static __global__ void step_tables_batched(const TableArgs* targs) {
  step_tables_body(targs[blockIdx.y], long(blockIdx.x) * blockDim.x + threadIdx.x);
}

// Set a flag when any field value is not finite (the step-size hazard of
// Sec. 3.2: a too-large dz makes the nonlinear increment blow up).
// exp(i m(x, y) Psi(z_n + o dz)) for the five distinct stage offsets
// o = 0, 1/4, 1/2, 3/4, 1 of steps n0 .. n0 + count - 1 (the first half-step
// uses offsets 0..2, the second 2..4), from the FP64 map and Psi reduced
// mod 2 pi in FP64.  Psi(z_n + o dz) = Psi_n + s_n o dz with Psi_n = psi0[n]
// and s_n = scale[n], or n dz and 1 without a scale profile.
struct MapArgs {
  const double* map;    // [ny][nx]
  const double* psi0;   // Psi_n prefix (NULL: no scale profile)
  const double* scale;  // s_n (NULL: no scale profile)
  float2* out;          // [count][5][ny][nx]
  unsigned plane;
  long long n0;              // first step (unless n0_dev is set)
  const long long* n0_dev;   // device copy of n0 (graph replays), or null
  double dz;
};

static __global__ void map_phase_table(MapArgs a) {
  const unsigned i = blockIdx.x * blockDim.x + threadIdx.x;
  if (i >= a.plane) return;
  const long long n = (a.n0_dev != nullptr ? *a.n0_dev : a.n0) + blockIdx.y;
  const double psi_n = a.psi0 != nullptr ? a.psi0[n] : double(n) * a.dz;
  const double s_n = a.scale != nullptr ? a.scale[n] : 1.0;
  const double m = a.map[i];
  float2* out = a.out + size_t(blockIdx.y) * 5 * a.plane;
  for (int k = 0; k < 5; ++k) {
    double sn, cs;
    phase_sincos(m * (psi_n + s_n * (0.25 * k) * a.dz), &sn, &cs);
    out[k * a.plane + i] = make_float2(float(cs), float(sn));
  }
}

// First step index of a chunk and the last step of the run (merged halves),
// for tables read by a replayed graph.
static __global__ void set_step_index(long long* dst, long long n0, long long merge_last) {
  if (blockIdx.x == 0 && threadIdx.x == 0) {
    dst[0] = n0;
    dst[1] = merge_last;
  }
}

static __global__ void finite_check(const float2* f, long n, int* flag) {
  long i = long(blockIdx.x) * blockDim.x + threadIdx.x;
  const long stride = long(gridDim.x) * blockDim.x;
  int bad = 0;
  for (; i < n; i += stride) {
    const float2 v = f[i];
    bad |= !(isfinite(v.x) && isfinite(v.y));
  }
  if (bad) atomicOr(flag, 1);
}

}  // namespace brahms
