// Batched recurrent decode step (Sec. 3.3): state <- lambda state + x_t,
// y_t = Re sum_m c state, for every (b, d) at once.
//
// A block covers 4 consecutive channels x 64 batch rows.  The block's 4*M
// (channel, mode) constants are computed once in float64 and split into a
// float32 pair lambda = hi + lo, so that a long run of steps does not drift by
// the rounding of a single float32 pole.  Each thread owns one (b, d): its M
// complex modes (M*8 bytes, contiguous) stay in registers for the update.
#include "common.h"
#include "kernels.h"

namespace res {

constexpr int DEC_CH = 4;
constexpr int DEC_ROWS = 64;

// Compiler-level ordering of the LDS accesses of one wave (the LDS executes a
// wave's accesses in program order).
__device__ __forceinline__ void wave_order() { asm volatile("" ::: "memory"); }

// One mode's update h <- (hi + lo) h + x and its readout term, with explicit
// fused multiply-adds so that every decode kernel rounds alike.
__device__ __forceinline__ float2 mode_step(float2 h, float2 hi, float2 lo, float xv) {
  const float tx = fmaf(lo.x, h.x, -(lo.y * h.y));
  const float ty = fmaf(lo.x, h.y, lo.y * h.x);
  return make_float2(fmaf(hi.x, h.x, fmaf(-hi.y, h.y, tx + xv)), fmaf(hi.x, h.y, fmaf(hi.y, h.x, ty)));
}
__device__ __forceinline__ float mode_readout(float2 c, float2 hn, float yv) {
  return fmaf(c.x, hn.x, fmaf(-c.y, hn.y, yv));
}

// The decode constants of one (channel, mode): lambda = exp(-gamma) e^{i omega}
// in float64, split into float32 hi + lo, and c = a e^{i phi}.  Every decode
// kernel and the constants table take them from here, so they agree bitwise.
__device__ __forceinline__ void decode_consts(float g32, float w32, float a32, float p32, float2& hi, float2& lo,
                                              float2& c) {
  const double g = g32, w = w32, a = a32, ph = p32;
  double s, co;
  sincos(w, &s, &co);
  const double e = exp(-g);
  const double lr = e * co, lim = e * s;
  hi = make_float2((float)lr, (float)lim);
  lo = make_float2((float)(lr - (double)hi.x), (float)(lim - (double)hi.y));
  sincos(ph, &s, &co);
  c = make_float2((float)(a * co), (float)(a * s));
}

template <typename TX, typename TY, int MF>
__global__ __launch_bounds__(DEC_CH* DEC_ROWS) void decode_kernel(
    const TX* __restrict__ x, TY* __restrict__ y, int B, int D, int M,
    const float* __restrict__ gamma, const float* __restrict__ omega,
    const float* __restrict__ amp, const float* __restrict__ phase, float* __restrict__ state) {
  __shared__ float2 lhi[DEC_CH][RES_M_MAX_DEV], llo[DEC_CH][RES_M_MAX_DEV], cs[DEC_CH][RES_M_MAX_DEV];
  const int tid = threadIdx.x;
  const int d0 = blockIdx.x * DEC_CH;
  const int b0 = blockIdx.y * DEC_ROWS;
  // MF > 0: M == MF is known, and the thread's state (MF complex modes) and
  // drive are loaded before the constants are computed, so their latency
  // overlaps that work
  float4 hv[MF > 0 ? MF / 2 : 1];
  float xf = 0.f;
  if (MF > 0) {
    const int dlf = tid % DEC_CH, bf = b0 + tid / DEC_CH, df = d0 + dlf;
    if (bf < B && df < D) {
      const size_t rowf = (size_t)bf * D + df;
      xf = to_f32(x[rowf]);
      const float4* sv = reinterpret_cast<const float4*>(state) + rowf * (MF / 2);
#pragma unroll
      for (int i = 0; i < MF / 2; ++i) hv[i] = sv[i];
    }
  }
  for (int t = tid; t < DEC_CH * M; t += blockDim.x) {
    const int dl = t / M, m = t % M, d = d0 + dl;
    float2 hi = make_float2(0.f, 0.f), lo = hi, c = hi;
    if (d < D) decode_consts(gamma[d * M + m], omega[d * M + m], amp[d * M + m], phase[d * M + m], hi, lo, c);
    lhi[dl][m] = hi;
    llo[dl][m] = lo;
    cs[dl][m] = c;
  }
  __syncthreads();
  const int dl = tid % DEC_CH;
  const int b = b0 + tid / DEC_CH;
  const int d = d0 + dl;
  if (b >= B || d >= D) return;
  const size_t row = (size_t)b * D + d;
  float yv = 0.f;
  if (MF > 0) {
    float4* sv = reinterpret_cast<float4*>(state) + row * (MF / 2);
#pragma unroll
    for (int i = 0; i < MF / 2; ++i) {
      float h[4] = {hv[i].x, hv[i].y, hv[i].z, hv[i].w};
      float hn[4];
#pragma unroll
      for (int j = 0; j < 2; ++j) {
        const int m = 2 * i + j;
        const float2 r = mode_step(make_float2(h[2 * j], h[2 * j + 1]), lhi[dl][m], llo[dl][m], xf);
        hn[2 * j] = r.x;
        hn[2 * j + 1] = r.y;
        yv = mode_readout(cs[dl][m], r, yv);
      }
      sv[i] = make_float4(hn[0], hn[1], hn[2], hn[3]);
    }
    y[row] = from_f32<TY>(yv);
    return;
  }
  const float xv = to_f32(x[row]);
  float2* st = reinterpret_cast<float2*>(state) + row * M;
  for (int m = 0; m < M; ++m) {
    const float2 hn = mode_step(st[m], lhi[dl][m], llo[dl][m], xv);
    st[m] = hn;
    yv = mode_readout(cs[dl][m], hn, yv);
  }
  y[row] = from_f32<TY>(yv);
}

template <typename TX, typename TY>
hipError_t launch_decode(int64_t B, int64_t D, int64_t M, const void* x, void* y,
                         const float* gamma, const float* omega, const float* amp,
                         const float* phase, float* state, hipStream_t st) {
  const dim3 grid((unsigned)((D + DEC_CH - 1) / DEC_CH), (unsigned)((B + DEC_ROWS - 1) / DEC_ROWS));
  if (M == 8 && ((uintptr_t)state & 15) == 0)  // 16-byte state loads
    hipLaunchKernelGGL((decode_kernel<TX, TY, 8>), grid, dim3(DEC_CH * DEC_ROWS), 0, st,
                       reinterpret_cast<const TX*>(x), reinterpret_cast<TY*>(y), (int)B, (int)D,
                       (int)M, gamma, omega, amp, phase, state);
  else
    hipLaunchKernelGGL((decode_kernel<TX, TY, 0>), grid, dim3(DEC_CH * DEC_ROWS), 0, st,
                       reinterpret_cast<const TX*>(x), reinterpret_cast<TY*>(y), (int)B, (int)D,
                       (int)M, gamma, omega, amp, phase, state);
  return hipGetLastError();
}

template hipError_t launch_decode<float, float>(int64_t, int64_t, int64_t, const void*, void*,
                                                const float*, const float*, const float*,
                                                const float*, float*, hipStream_t);
template hipError_t launch_decode<bf16_t, bf16_t>(int64_t, int64_t, int64_t, const void*, void*,
                                                  const float*, const float*, const float*,
                                                  const float*, float*, hipStream_t);
template hipError_t launch_decode<bf16_t, float>(int64_t, int64_t, int64_t, const void*, void*,
                                                 const float*, const float*, const float*,
                                                 const float*, float*, hipStream_t);

// ---------------------------------------------------------------------------
// Decode from a constants table.  resonator_decode_constants evaluates the
// constants of every (channel, mode) once (decode_consts) into
// tab[d][m] = (hi.re, hi.im, lo.re, lo.im, c.re, c.im); the step kernel then
// reads them instead of evaluating float64 exp and sincos per call.  A work-group
// is one wave: 64 consecutive channels of one batch row (each thread one (b, d),
// its modes in registers), so the wave's state (4 KB at M = 8), constants and
// drive and output rows are contiguous; a step over B x D needs B D / 64
// work-groups (256 at B64 D256).  The arithmetic and its order are
// decode_kernel's, so a step from the table gives the bits of
// resonator_decode_step.
// ---------------------------------------------------------------------------
constexpr int DTB_CH = 64;
constexpr int DTB_ROWS = 1;

__global__ void decode_consts_kernel(int D, int M, const float* __restrict__ gamma, const float* __restrict__ omega,
                                     const float* __restrict__ amp, const float* __restrict__ phase,
                                     float* __restrict__ tab) {
  const int i = blockIdx.x * blockDim.x + threadIdx.x;
  if (i >= D * M) return;
  float2 hi, lo, c;
  decode_consts(gamma[i], omega[i], amp[i], phase[i], hi, lo, c);
  float2* t = reinterpret_cast<float2*>(tab) + (size_t)i * 3;
  t[0] = hi;
  t[1] = lo;
  t[2] = c;
}

hipError_t launch_decode_consts(int64_t D, int64_t M, const float* gamma, const float* omega, const float* amp,
                                const float* phase, float* tab, hipStream_t st) {
  const int n = (int)(D * M);
  hipLaunchKernelGGL(decode_consts_kernel, dim3((unsigned)((n + 255) / 256)), dim3(256), 0, st, (int)D, (int)M,
                     gamma, omega, amp, phase, tab);
  return hipGetLastError();
}

template <typename TX, typename TY, int MF>
__global__ __launch_bounds__(DTB_CH* DTB_ROWS) void decode_tab_kernel(const TX* __restrict__ x,
                                                                     TY* __restrict__ y, int B, int D, int M,
                                                                     const float* __restrict__ tab,
                                                                     float* __restrict__ state) {
  const int tid = threadIdx.x;
  const int dl = tid % DTB_CH;
  const int b = blockIdx.y * DTB_ROWS + tid / DTB_CH;
  const int d = blockIdx.x * DTB_CH + dl;
  if (b >= B || d >= D) return;
  const size_t row = (size_t)b * D + d;
  const float2* t = reinterpret_cast<const float2*>(tab) + (size_t)d * M * 3;
  float yv = 0.f;
  if (MF > 0) {
    // all loads first: drive, state (16-byte pieces), constants
    const float xv = to_f32(x[row]);
    float4* sv = reinterpret_cast<float4*>(state) + row * (MF / 2);
    const float4* tv = reinterpret_cast<const float4*>(t);
    float4 hv[MF > 0 ? MF / 2 : 1], cv[MF > 0 ? MF * 3 / 2 : 1];
#pragma unroll
    for (int i = 0; i < MF / 2; ++i) hv[i] = sv[i];
#pragma unroll
    for (int i = 0; i < MF * 3 / 2; ++i) cv[i] = tv[i];
    const float* cf = reinterpret_cast<const float*>(cv);
#pragma unroll
    for (int i = 0; i < MF / 2; ++i) {
      float h[4] = {hv[i].x, hv[i].y, hv[i].z, hv[i].w};
      float hn[4];
#pragma unroll
      for (int j = 0; j < 2; ++j) {
        const int m = 2 * i + j;
        const float* k = cf + 6 * m;
        const float2 r = mode_step(make_float2(h[2 * j], h[2 * j + 1]), make_float2(k[0], k[1]),
                                   make_float2(k[2], k[3]), xv);
        hn[2 * j] = r.x;
        hn[2 * j + 1] = r.y;
        yv = mode_readout(make_float2(k[4], k[5]), r, yv);
      }
      sv[i] = make_float4(hn[0], hn[1], hn[2], hn[3]);
    }
    y[row] = from_f32<TY>(yv);
    return;
  }
  const float xv = to_f32(x[row]);
  float2* st = reinterpret_cast<float2*>(state) + row * M;
  for (int m = 0; m < M; ++m) {
    const float2 hn = mode_step(st[m], t[3 * m], t[3 * m + 1], xv);
    st[m] = hn;
    yv = mode_readout(t[3 * m + 2], hn, yv);
  }
  y[row] = from_f32<TY>(yv);
}

template <typename TX, typename TY>
hipError_t launch_decode_tab(int64_t B, int64_t D, int64_t M, const void* x, void* y, const float* tab,
                             float* state, hipStream_t st) {
  const dim3 grid((unsigned)((D + DTB_CH - 1) / DTB_CH), (unsigned)((B + DTB_ROWS - 1) / DTB_ROWS));
  if (M == 8 && ((uintptr_t)state & 15) == 0 && ((uintptr_t)tab & 15) == 0)  // 16-byte loads
    hipLaunchKernelGGL((decode_tab_kernel<TX, TY, 8>), grid, dim3(DTB_CH * DTB_ROWS), 0, st,
                       reinterpret_cast<const TX*>(x), reinterpret_cast<TY*>(y), (int)B, (int)D, (int)M, tab,
                       state);
  else
    hipLaunchKernelGGL((decode_tab_kernel<TX, TY, 0>), grid, dim3(DTB_CH * DTB_ROWS), 0, st,
                       reinterpret_cast<const TX*>(x), reinterpret_cast<TY*>(y), (int)B, (int)D, (int)M, tab,
                       state);
  return hipGetLastError();
}
#define RES_DECODE_TAB_INST(TX, TY)                                                                      \
  template hipError_t launch_decode_tab<TX, TY>(int64_t, int64_t, int64_t, const void*, void*, const float*, \
                                                float*, hipStream_t);
RES_DECODE_TAB_INST(float, float)
RES_DECODE_TAB_INST(bf16_t, bf16_t)
RES_DECODE_TAB_INST(bf16_t, float)
#undef RES_DECODE_TAB_INST

// ---------------------------------------------------------------------------
// Several decode steps in one launch, for drives known in advance (a prompt
// chunk, drafted tokens to verify, a captured block of tokens).  Step n applies
// the update and readout of decode_kernel with the same constants and in the
// same order, so N steps here give the same bits as N single steps.
//
// What bounds it is each mode's chain of dependent steps, so the modes of a
// (b, d) are spread over R = 8 or 16 lanes, one mode each (B64 D256 M8: 2048
// waves, two per SIMD; one thread per (b, d) leaves three of four SIMDs idle:
// 128 steps 52 us, now 17).  The readout needs a
// step's modes in their order: the lanes take R steps, leave every step's states
// in LDS, and lane r then reads out step r with all its modes, so the readout
// is spread over the lanes by step.  Lane r also loads step r's drive, one
// batch of R steps ahead.  All exchange stays inside a wave (no barrier in the
// step loop).
//
// A block is CH channels x DMS_ROWS batch rows (one wave per row).  The up to
// DMS_XCD blocks of neighbouring channels that share the 128-byte lines of a
// row's drives and outputs are 8 apart in the grid, which the dispatcher places
// on one XCD (work-groups go round-robin over the 8 XCDs).  Narrow inputs have
// smaller groups, so that no block starts only to end (B4096 D16: 10 us with
// groups of 8, of which 2 had work).
// ---------------------------------------------------------------------------
constexpr int DMS_ROWS = 4;  // waves of a block
constexpr int DMS_XCD = 8;

// log2 of the blocks of a group, for a row of D channels in blocks of ch: a power of
// two up to DMS_XCD (shifts in the kernel: divisions by it cost 0.6 us at B160 D256)
inline int dms_group(int64_t D, int ch) {
  int lx = 0;
  while ((1 << lx) < DMS_XCD && (int64_t)ch << lx < D) ++lx;
  return lx;
}

template <typename TX, typename TY, int R>
__global__ __launch_bounds__(64 * DMS_ROWS) void decode_steps_kernel(
    const TX* __restrict__ x, TY* __restrict__ y, int B, int64_t N, int D, int M, int lx, int64_t sn, int64_t sb,
    const float* __restrict__ gamma, const float* __restrict__ omega, const float* __restrict__ amp,
    const float* __restrict__ phase, float* __restrict__ state) {
  constexpr int CH = 64 / R;         // channels of a block
  constexpr int HROW = R + 2;        // float2 per step row of the states (16 bytes of bank offset)
  constexpr int HGRP = R * HROW + 8; // float2 per (b, d)
  __shared__ float2 lhi[64], llo[64], cs[64];
  __shared__ __align__(16) float xs[DMS_ROWS * CH][R];
  __shared__ __align__(16) float2 hs[DMS_ROWS * CH * HGRP];
  const int lane = threadIdx.x & 63, wave = threadIdx.x >> 6;
  const int m = lane % R, cl = lane / R;
  // block -> (row block, channel block): member k of a group of 2^lx channel
  // blocks, groups over channels then rows
  const unsigned bid = blockIdx.x;
  const unsigned grp = (bid >> (3 + lx)) * 8 + (bid & 7);
  const unsigned ngd = (unsigned)(D + (CH << lx) - 1) >> ((R == 8 ? 3 : 2) + lx);
  const unsigned gr = grp / ngd;
  const int d0 = (int)(((grp - gr * ngd) << lx) + ((bid >> 3) & ((1u << lx) - 1))) * CH;
  const int64_t b0 = (int64_t)gr * DMS_ROWS;
  if (d0 >= D || b0 >= B) return;  // the whole block
  const int64_t b = b0 + wave;
  const int d = d0 + cl;
  const bool valid = b < B && d < D;
  const int64_t bc = b < B ? b : B - 1;
  const int dc = d < D ? d : D - 1;
  // the state and the first R drives load while the constants are evaluated
  float2* st = reinterpret_cast<float2*>(state) + ((size_t)bc * D + dc) * M;
  float2 h = make_float2(0.f, 0.f);
  if (m < M) h = st[m];
  const int64_t xo = bc * sb + dc;
  TX xn = x[(m < N ? (int64_t)m : N - 1) * sn + xo];
  if (threadIdx.x < 64) {
    float2 hi = make_float2(0.f, 0.f), lo = hi, c = hi;
    if (d < D && m < M) {
      const int i = d * M + m;
      decode_consts(gamma[i], omega[i], amp[i], phase[i], hi, lo, c);
    }
    lhi[lane] = hi;
    llo[lane] = lo;
    cs[lane] = c;
  }
  __syncthreads();
  const float2 hi = lhi[lane], lo = llo[lane];
  float2 c[R];
#pragma unroll
  for (int k = 0; k < R; ++k) c[k] = cs[cl * R + k];
  float* xg = xs[wave * CH + cl];
  float2* hg = hs + (size_t)(wave * CH + cl) * HGRP;
  for (int64_t n0 = 0; n0 < N; n0 += R) {
    xg[m] = to_f32(xn);
    {  // past the last step the index is clamped to it and the value is not used
      const int64_t nn = n0 + R + m;
      xn = x[(nn < N ? nn : N - 1) * sn + xo];
    }
    wave_order();
    const int nr = N - n0 < R ? (int)(N - n0) : R;
    float xv[R];
#pragma unroll
    for (int j = 0; j < R; j += 4) {
      const float4 v = *reinterpret_cast<const float4*>(xg + j);
      xv[j] = v.x;
      xv[j + 1] = v.y;
      xv[j + 2] = v.z;
      xv[j + 3] = v.w;
    }
#pragma unroll
    for (int j = 0; j < R; ++j) {
      if (j < nr) {
        h = mode_step(h, hi, lo, xv[j]);
        hg[j * HROW + m] = h;
      }
    }
    wave_order();
    float yv = 0.f;
    const float4* hr = reinterpret_cast<const float4*>(hg + m * HROW);
#pragma unroll
    for (int k = 0; k < R; k += 2) {
      const float4 v = hr[k / 2];
      if (k < M) yv = mode_readout(c[k], make_float2(v.x, v.y), yv);
      if (k + 1 < M) yv = mode_readout(c[k + 1], make_float2(v.z, v.w), yv);
    }
    if (valid && m < nr) y[(n0 + m) * sn + xo] = from_f32<TY>(yv);
    wave_order();
  }
  if (valid && m < M) st[m] = h;
}

// The same steps for many (b, d): a thread owns one (b, d) and keeps its M modes
// in registers for all N steps; a wave covers 64 consecutive channels of one
// batch row, so every step's drive and output rows are coalesced, and the next
// step's drive is loaded before the current step is computed.  With enough
// waves to fill the SIMDs it needs no exchange and is the faster one.
constexpr int DMW_CH = 64;
constexpr int DMW_ROWS = 4;
// Whether one thread per pair is the faster of the two.  Above 65536 pairs it is
// (128 steps, M = 8: at 65536 pairs 55 us against 38 with a lane per mode, at
// 131072 58 against 65, at 262144 92 against 125; M = 2: 37 against 46 at 98304).
// Below, the times of both follow these fits (us; bf16, 16000 to 65536 pairs, M 1
// to 16, 1 to 64 steps; within 10 % where the two are close).  A lane per mode:
// the work is its waves' (kw thousand), idle lanes (M < R) among them.  A thread
// per pair: the latency of M modes in turn, more where a narrow D leaves lanes
// idle and so more than two thousand waves.  At 65536 pairs of 256 channels, a
// lane per mode against a thread per pair: M = 1 one step 6.4, 4.4, 64 steps 21.0,
// 17.9; M = 4 8 steps 7.5, 7.0, 64 steps 21.4, 22.6; M = 8 one step 7.2, 8.3; M = 9
// one step 14.0, 10.3.
static bool steps_wide(int64_t B, int64_t D, int64_t M, int64_t N) {
  if (B * D > (1 << 16)) return true;
  const int R = M <= 8 ? 8 : 16, ch = 64 / R;
  const bool bank = M > 8;
  const double m = (double)M, n = (double)(N - 1), kw = (double)((D + ch - 1) / ch * B) / 1024;
  const double lane = bank ? 2.6 + 0.72 * kw + n * kw * (N <= 16 ? 0.018 : 0.0255)
                           : 3.8 + 0.22 * kw + (kw > 7 ? 0.8 : 0.0) + n * (kw > 3.3 ? 0.027 * kw : 0.09);
  const double ww = (double)((D + DMW_CH - 1) / DMW_CH * B) / 1024, over = ww > 2 ? ww - 2 : 0;
  const double base = D < DMW_CH ? 4.2 + 0.36 * m : M <= 4 ? 4.0 + 0.3 * m : bank ? 5.0 + 0.5 * m : 4.0 + 0.45 * m;
  const double step = bank ? (0.14 + 0.045 * m) * (1 + 0.47 * over) : (0.18 + 0.025 * m) * (1 + 0.21 * over);
  return base + over * (bank ? 2.6 : 0.6) + n * step < lane;
}

// ROWS: batch-major strides formed here from N and D (16 modes, 98304 pairs, 64
// steps: 61 us against 64 with the given ones; 8 modes the given ones: 22.0 against
// 23.0 at M = 3).
template <typename TX, typename TY, int MM, bool ROWS>
__global__ __launch_bounds__(DMW_CH* DMW_ROWS) void decode_steps_wide_kernel(
    const TX* __restrict__ x, TY* __restrict__ y, int B, int64_t N, int D, int M, int64_t sn, int64_t sb,
    const float* __restrict__ gamma, const float* __restrict__ omega, const float* __restrict__ amp,
    const float* __restrict__ phase, float* __restrict__ state) {
  __shared__ float2 lhi[DMW_CH][MM], llo[DMW_CH][MM], cs[DMW_CH][MM];
  const int tid = threadIdx.x;
  const int d0 = blockIdx.x * DMW_CH;
  const int b0 = (int)(blockIdx.z * gridDim.y + blockIdx.y) * DMW_ROWS;  // over two dimensions: any B
  if (ROWS) {
    sn = D;
    sb = N * D;
  }
  for (int t = tid; t < DMW_CH * M; t += blockDim.x) {
    const int dl = t / M, m = t % M, d = d0 + dl;
    float2 hi = make_float2(0.f, 0.f), lo = hi, c = hi;
    if (d < D) decode_consts(gamma[d * M + m], omega[d * M + m], amp[d * M + m], phase[d * M + m], hi, lo, c);
    lhi[dl][m] = hi;
    llo[dl][m] = lo;
    cs[dl][m] = c;
  }
  __syncthreads();
  const int dl = tid % DMW_CH;
  const int b = b0 + tid / DMW_CH;
  const int d = d0 + dl;
  if (b >= B || d >= D) return;  // no barrier follows
  float2 h[MM], hi[MM], lo[MM], c[MM];
  float2* st = reinterpret_cast<float2*>(state) + ((size_t)b * D + d) * M;
#pragma unroll
  for (int m = 0; m < MM; ++m) {
    if (m < M) {
      h[m] = st[m];
      hi[m] = lhi[dl][m];
      lo[m] = llo[dl][m];
      c[m] = cs[dl][m];
    }
  }
  const TX* xr = x + (size_t)b * sb + d;
  TY* yr = y + (size_t)b * sb + d;
  // Drives of the next DPF steps are loaded while the current DPF are computed.
  // Past the last step the index is clamped to it (the value is not used), so
  // the loads are unconditional and none waits behind a branch.
  constexpr int DPF = 8;
  TX xb[DPF];
#pragma unroll
  for (int j = 0; j < DPF; ++j) xb[j] = xr[(j < N ? (int64_t)j : N - 1) * sn];
  for (int64_t n0 = 0; n0 < N; n0 += DPF) {
    TX xn[DPF];
#pragma unroll
    for (int j = 0; j < DPF; ++j) {
      const int64_t nn = n0 + DPF + j;
      xn[j] = xr[(nn < N ? nn : N - 1) * sn];
    }
#pragma unroll
    for (int j = 0; j < DPF; ++j) {
      if (n0 + j < N) {
        float yv = 0.f;
#pragma unroll
        for (int m = 0; m < MM; ++m) {
          if (m < M) {
            h[m] = mode_step(h[m], hi[m], lo[m], to_f32(xb[j]));
            yv = mode_readout(c[m], h[m], yv);
          }
        }
        yr[(n0 + j) * sn] = from_f32<TY>(yv);
      }
    }
#pragma unroll
    for (int j = 0; j < DPF; ++j) xb[j] = xn[j];
  }
#pragma unroll
  for (int m = 0; m < MM; ++m)
    if (m < M) st[m] = h[m];
}

template <typename TX, typename TY>
hipError_t launch_decode_steps(int64_t B, int64_t N, int64_t D, int64_t M, const void* x, void* y, bool time_major,
                               const float* gamma, const float* omega, const float* amp,
                               const float* phase, float* state, hipStream_t st) {
  const int64_t sn = time_major ? B * D : D, sb = time_major ? D : N * D;
  // One step of many pairs with a wide bank: the single-step kernel, whose states
  // load 16 bytes at a time or stream through one mode at a time (M = 8, 1048576
  // pairs: 38 us against 49, M = 16 75 against 129; M <= 2 is slower there, 18
  // against 16, and M = 6 38 against 35)
  if (N == 1 && M >= 8 && B * D > (1 << 16) && B <= DEC_ROWS * 65535LL)
    return launch_decode<TX, TY>(B, D, M, x, y, gamma, omega, amp, phase, state, st);
  if (steps_wide(B, D, M, N)) {
    const int64_t nb = (B + DMW_ROWS - 1) / DMW_ROWS, gy = nb < 65535 ? nb : 65535;
    const dim3 wgrid((unsigned)((D + DMW_CH - 1) / DMW_CH), (unsigned)gy, (unsigned)((nb + gy - 1) / gy));
    const auto kernel = M <= 8       ? decode_steps_wide_kernel<TX, TY, 8, false>
                        : time_major ? decode_steps_wide_kernel<TX, TY, RES_M_MAX_DEV, false>
                                     : decode_steps_wide_kernel<TX, TY, RES_M_MAX_DEV, true>;
    hipLaunchKernelGGL(kernel, wgrid, dim3(DMW_CH * DMW_ROWS), 0, st, reinterpret_cast<const TX*>(x),
                       reinterpret_cast<TY*>(y), (int)B, N, (int)D, (int)M, sn, sb, gamma, omega, amp, phase, state);
    return hipGetLastError();
  }
  const int R = M <= 8 ? 8 : 16;
  const int lx = dms_group(D, 64 / R);
  const int64_t gch = (int64_t)(64 / R) << lx;  // channels of a group of blocks
  const int64_t groups = (D + gch - 1) / gch * ((B + DMS_ROWS - 1) / DMS_ROWS);
  const dim3 grid((unsigned)((groups + 7) / 8 * 8 << lx)), block(64 * DMS_ROWS);
  if (R == 8)
    hipLaunchKernelGGL((decode_steps_kernel<TX, TY, 8>), grid, block, 0, st, reinterpret_cast<const TX*>(x),
                       reinterpret_cast<TY*>(y), (int)B, N, (int)D, (int)M, lx, sn, sb, gamma, omega, amp, phase,
                       state);
  else
    hipLaunchKernelGGL((decode_steps_kernel<TX, TY, 16>), grid, block, 0, st, reinterpret_cast<const TX*>(x),
                       reinterpret_cast<TY*>(y), (int)B, N, (int)D, (int)M, lx, sn, sb, gamma, omega, amp, phase,
                       state);
  return hipGetLastError();
}

#define RES_DECODE_STEPS_INST(TX, TY)                                                                   \
  template hipError_t launch_decode_steps<TX, TY>(int64_t, int64_t, int64_t, int64_t, const void*, void*, \
                                                  bool, const float*, const float*, const float*,       \
                                                  const float*, float*, hipStream_t);
RES_DECODE_STEPS_INST(float, float)
RES_DECODE_STEPS_INST(bf16_t, bf16_t)
RES_DECODE_STEPS_INST(bf16_t, float)
#undef RES_DECODE_STEPS_INST

}  // namespace res
