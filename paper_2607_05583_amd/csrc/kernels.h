// Internal launch interface between the C ABI (api.hip) and the kernel files.
#pragma once

#include <hip/hip_ext.h>

#include "common.h"

namespace res {

// Mixer epilogue: limits and the block of rows of the parameter sums
constexpr int EPI_H_MAX = 32;   // heads
constexpr int EPI_K_MAX = 16;   // local-path taps
constexpr int EPI_ROWS = 64;    // rows per block partial
// Workspace of the epilogue backward: rows of block partials (one per work-group
// of the parameter sums), then H*H float64 terms.  The generic kernels write one
// row per EPI_ROWS rows of activations; the tile kernel as many as it has
// work-groups (at most EPI_PARTS: three on each of 256 compute units).
constexpr int64_t EPI_PARTS = 768;
inline int64_t epi_part_cols(int64_t H, int64_t dh, int64_t K) { return H * H + H * dh + H * dh * K; }
inline int64_t epi_part_rows_min(int64_t B, int64_t L) { return B * ((L + EPI_ROWS - 1) / EPI_ROWS); }
inline size_t epi_bytes_of_rows(int64_t rows, int64_t H, int64_t dh, int64_t K) {
  const int64_t f = (rows * epi_part_cols(H, dh, K) + 1) & ~(int64_t)1;  // even: the float64 terms are 8-byte aligned
  return (size_t)f * sizeof(float) + (size_t)(H * H) * sizeof(double);
}
// the least workspace a call takes, and what the query returns
inline size_t epi_workspace_min(int64_t B, int64_t L, int64_t H, int64_t dh, int64_t K) {
  return epi_bytes_of_rows(epi_part_rows_min(B, L), H, dh, K);
}
inline size_t epi_workspace_bytes(int64_t B, int64_t L, int64_t H, int64_t dh, int64_t K) {
  const int64_t least = epi_part_rows_min(B, L);
  return epi_bytes_of_rows(least > EPI_PARTS ? least : EPI_PARTS, H, dh, K);
}

// Three-kernel forward (M > 8, or more chains than the single-pass one counts).
struct FwdArgs {
  const void* x;
  void* y;
  int64_t B, L;
  int D, M;
  int NB, Dp, Mp;
  int64_t P;
  int last_len;
  int fast_io;       // x and y 16-byte aligned and D * element size a multiple of 16
  const void* tab;
  const ModeScalars* scal;
  const ModeCarry* cc;
  const float* h0;   // [B][D][M][2] or null
  float* h_out;      // [B][D][M][2] or null: state at t = L-1
  void* agg;         // per tile [DW * Mp] float4: half-tile end states (A_0, A_1)
  void* car;         // per tile [DW * Mp] float4: entry states of both halves
  float2* alast;     // [B][Dp][Mp]: state at t = L-1 from a zero start at the last tile
};

// First of a chain's four counter words (65536 chains in all).  The first 4096
// chains have 256 bytes to themselves: the arrivals and decisions of a chain's
// work-groups are atomics on one line each, and with 16 chains on two lines (B4
// D256 bf16) the 256 work-groups passed after 10 instead of 6.6 thousand cycles.
__host__ __device__ inline size_t stream_chain_word(int chain) {
  return 64 * (size_t)(chain & 4095) + 4 * (size_t)(chain >> 12);
}

// Single-pass forward (M <= 8): problem, parameters and the workspace regions.
// A published segment state is a set of 64-bit words, each a float (low half)
// and the call's tag, epoch + 1 (high half); hdr[1] holds the epoch.
struct StreamArgs {
  const void* x;
  void* y;
  int64_t B, L;
  int D, M;
  int NB;              // channel blocks of DW channels
  int nchains;         // B * NB
  int G, Sf, Sr;       // work-groups of a chain; its tiles over them, quotient and remainder
  int64_t P;           // tiles per chain
  int last_len;        // valid steps of a chain's last tile
  int fast_io;         // x and y 16-byte aligned and rows a multiple of 16 bytes
  const float* gamma;
  const float* omega;
  const float* amp;
  const float* phase;
  const float* h0;     // [B][D][M][2] or null
  float* h_out;        // [B][D][M][2] or null
  uint32_t* hdr;       // [0] status (bit 0: a wait gave up, bit 1: stale counters), [1] epoch,
                       // [2] finished chains, [4] a wait of this call gave up
  uint32_t* chainw;    // [65536][4] (stream_chain_word): next ticket, arrived work-groups, segment order (0 open,
                       // 1 static, 2 tickets), finished work-groups
  uint64_t* agg;       // [nchains][G][DW / 4 waves][64] published state of each segment
                       // (float | tag << 32 per word); laid out for up to P segments.  The
                       // prompt state: [nchains][G][DW][modes] complex float64 end states
};

// Backward (M <= 16).  A chain is one batch row and one block of DW channels
// (64-byte rows: 32 bf16 or 16 float channels), cut into nseg segments of S
// tiles (the last may be shorter), one work-group per segment.
struct BwdArgs {
  const void* x;
  const void* dy;
  void* dx;
  int64_t B, L;
  int D, M;
  int NB;               // channel blocks of the backward
  int Dp, Mp;           // padded channels and modes (record strides)
  int64_t P;            // tiles per row
  int64_t S;            // tiles per segment
  int nseg;             // segments per row
  int64_t Ss;           // tiles per record segment (the record pass's own segmentation)
  int nss;              // record segments per row
  int sf;               // record segments per segment (S = sf Ss; 1 or 2)
  int fast_io;          // x, dy and dx 16-byte aligned and rows a multiple of 16 bytes
  const void* tab;
  const ModeScalars* scal;
  const ModeCarry* cc;
  float4* agg;          // [B][nss][Dp][Mp]: (Q, rho) of a record segment's own drives at its left edge
  float* part;          // [B][nseg][Dp][16 + 4 Mp]: partial sums of G, W and R per segment
  float4* q0;           // [B][Dp][Mp]: (Q, rho) at t = 0
};

template <typename TA>
hipError_t launch_prep(const Geometry& g, const float* gamma, const float* omega, const float* amp,
                       const float* phase, bool bwd, void* tab, ModeScalars* scal, ModeCarry* cc,
                       hipStream_t st);

template <typename TX>
hipError_t launch_fwd_agg(const Geometry& g, const FwdArgs& a, hipStream_t st,
                          hipEvent_t ev0 = nullptr, hipEvent_t ev1 = nullptr);

hipError_t launch_fwd_carry(const Geometry& g, const FwdArgs& a, hipStream_t st);

// Work-groups per call of the single-pass forward, and its launch.
template <typename TX>
hipError_t launch_state(const StreamArgs& a, hipStream_t st);
hipError_t launch_stream_init(uint32_t* hdr, uint32_t* chainw, void* agg, int nchains, size_t agg_bytes,
                              hipStream_t st);
// At most STREAM_GROUPS of them share chains (and publish states).
constexpr int STREAM_GROUPS = 256;
int fwd_stream_grid(int64_t nchains, int64_t P, int num_cus);
template <typename TX, typename TY>
hipError_t launch_fwd_stream(const StreamArgs& a, int grid, hipStream_t st, hipEvent_t ev0, hipEvent_t ev1);

template <typename TX, typename TY>
hipError_t launch_fwd_apply(const Geometry& g, const FwdArgs& a, hipStream_t st, hipEvent_t ev0,
                            hipEvent_t ev1);

// Launch with optional start/stop events recorded around this one kernel.
template <typename K, typename... Args>
inline void launch_timed(K kernel, dim3 grid, dim3 block, hipStream_t st, hipEvent_t ev0,
                         hipEvent_t ev1, Args... args) {
  if (ev0 != nullptr)
    hipExtLaunchKernelGGL(kernel, grid, block, 0, st, ev0, ev1, 0, args...);
  else
    hipLaunchKernelGGL(kernel, grid, block, 0, st, args...);
}

hipError_t launch_fill_zero(float* p, int64_t n, hipStream_t st);

template <typename TX, typename TY>
hipError_t launch_decode(int64_t B, int64_t D, int64_t M, const void* x, void* y,
                         const float* gamma, const float* omega, const float* amp,
                         const float* phase, float* state, hipStream_t st);
const char* launch_grouped_linear(const void* x, const void* W, void* y, int64_t N, int64_t d_in, int64_t d_out,
                                  int64_t G, bool bf16, hipStream_t st);
// MFMA grouped projection (proj.hip): one or two weights (W1 null for one) over
// the same x; shapes and alignments the kernel takes, else the library GEMM
bool grouped_proj_supported(const void* x, const void* W0, const void* W1, const void* y0, const void* y1,
                            int64_t d_in, int64_t d_out, int64_t G, bool bf16);
hipError_t launch_grouped_proj(const void* x, const void* W0, const void* W1, void* y0, void* y1, int64_t N,
                               int64_t d_in, int64_t d_out, int64_t G, bool bf16, int num_cus, hipStream_t st);
bool grouped_dgrad_supported(int n, const void* const* dy, const void* const* W, const void* dx, int64_t d_in,
                             int64_t d_out, int64_t G, bool bf16);
hipError_t launch_grouped_dgrad(int n, const void* const* dy, const void* const* W, void* dx, int64_t N, int64_t d_in,
                                int64_t d_out, int64_t G, bool bf16, bool accumulate, int num_cus, hipStream_t st);
int grouped_wgrad_blocks(int n, int nout, int64_t d_in, int64_t d_out, int64_t G, bool bf16);
int64_t grouped_wgrad_grid(int64_t N, int n);
hipError_t launch_grouped_wgrad(int n, const void* x, const void* const* dy, const int* out, float* dW0, float* dW1,
                                int64_t N, int64_t d_in, int64_t d_out, int64_t G, bool accumulate, float* part,
                                hipStream_t st);
const char* launch_grouped_linear_bwd_data(const void* dy, const void* W, void* dx, int64_t N, int64_t d_in,
                                           int64_t d_out, int64_t G, bool bf16, bool accumulate, hipStream_t st);
const char* launch_grouped_linear_bwd_weight(const void* x, const void* dy, float* dW, int64_t N, int64_t d_in,
                                             int64_t d_out, int64_t G, bool bf16, bool accumulate, hipStream_t st);
hipError_t launch_block_diag(const void* W, void* Wd, int64_t d_in, int64_t d_out, int64_t G, bool bf16,
                             hipStream_t st);
constexpr int64_t SPLITK_TARGET = 64;     // partial products of the split-K weight gradient
constexpr int64_t SPLITK_MIN_ROWS = 256;  // rows per partial at least
int64_t splitk_rows(int64_t N);
int64_t splitk_parts(int64_t N);
const char* launch_grouped_linear_bwd_weight_splitk(const void* x, const void* dy, float* dW, int64_t N,
                                                    int64_t d_in, int64_t d_out, int64_t G, bool bf16,
                                                    bool accumulate, float* P, hipStream_t st);
hipError_t launch_block_extract(const float* Wd, float* W, int64_t d_in, int64_t d_out, int64_t G, bool accumulate,
                                hipStream_t st);
size_t quad_workspace_bytes(int64_t L, int64_t D);
size_t fft_next_pow2(int64_t L);
const char* fft_workspace_bytes(int64_t B, int64_t L, int64_t D, size_t* bytes);
const char* launch_fft_reference(const float* x, float* y, int64_t B, int64_t L, int64_t D, int64_t M,
                                 const float* gamma, const float* omega, const float* amp, const float* phase,
                                 void* ws, hipStream_t st);
hipError_t launch_quad_reference(const float* x, float* y, int64_t B, int64_t L, int64_t D, int64_t M,
                                 const float* gamma, const float* omega, const float* amp, const float* phase,
                                 float* K, hipStream_t st);
hipError_t launch_params_map(const float* tg, const float* tw, int64_t n, float alpha_min, float* gamma,
                             float* omega, hipStream_t st);
hipError_t launch_params_map_bwd(const float* tg, const float* tw, const float* dg, const float* dw, int64_t n,
                                 float* dtg, float* dtw, hipStream_t st);
hipError_t launch_diagnostics(const float* gamma, const float* omega, const float* amp, const float* phase, int64_t D,
                              int64_t M, int64_t T, float* hl, float* en, float* spec, hipStream_t st);
hipError_t launch_params_init(int64_t D, int64_t M, double hl_min, double hl_max, double per_min, double per_max,
                              double alpha_min, float* tg, float* tw, hipStream_t st);
hipError_t launch_decode_consts(int64_t D, int64_t M, const float* gamma, const float* omega, const float* amp,
                                const float* phase, float* tab, hipStream_t st);
template <typename TX, typename TY>
hipError_t launch_decode_tab(int64_t B, int64_t D, int64_t M, const void* x, void* y, const float* tab,
                             float* state, hipStream_t st);
template <typename TX, typename TY>
hipError_t launch_decode_steps(int64_t B, int64_t N, int64_t D, int64_t M, const void* x, void* y, bool time_major,
                               const float* gamma, const float* omega, const float* amp,
                               const float* phase, float* state, hipStream_t st);

// Segments per row of the backward for a device of num_cus compute units.
int bwd_segments(int64_t nchains, int64_t P, int num_cus);
// Channels per block of the backward.
inline int bwd_block_channels(int elem_bytes) { return 64 / elem_bytes; }

template <typename TX>
hipError_t launch_bwd(const BwdArgs& a, hipStream_t st, hipEvent_t ev0 = nullptr, hipEvent_t ev1 = nullptr);

hipError_t launch_bwd_reduce(const Geometry& g, int nseg, const float* part, const float4* q0,
                             const ModeCarry* cc, const float* h0, float* dgamma, float* domega,
                             float* damp, float* dphase, float* dh0, hipStream_t st);

template <typename T>
hipError_t launch_epi_fwd(const void* y, const void* gate, const void* v, void* z, int64_t B, int64_t L, int H,
                          int dh, int K, const float* Ct, float lambda_c, const float* w, const float* s, int vec,
                          hipStream_t st);
// epilogue fused with the grouped output projection (one group per head)
size_t epi_proj_lds(int H, int dh, int K, int64_t d_out, bool bf16);
size_t epi_z_lds(int H, int dh, int K, bool bf16);
template <typename T>
hipError_t launch_epi_z_fwd(const void* y, const void* gate, const void* v, void* z, int64_t B, int64_t L, int H,
                            int K, const float* Ct, float lambda_c, const float* w, const float* s, int num_cus,
                            hipStream_t st);
template <typename T>
hipError_t launch_epi_proj_fwd(const void* y, const void* gate, const void* v, const void* Wo, void* out, void* z, int64_t B,
                               int64_t L, int H, int K, int64_t d_out, const float* Ct, float lambda_c,
                               const float* w, const float* s, int num_cus, hipStream_t st);
template <typename T>
hipError_t launch_epi_bwd(const void* y, const void* gate, const void* v, const void* dz, void* dy, void* dgate,
                          void* dv, int64_t B, int64_t L, int H, int dh, int K, const float* Ct, float lambda_c,
                          const float* w, const float* s, float* dCt, float* dlambda_c, float* dw, float* ds,
                          float* part, size_t ws_bytes, int vec, hipStream_t st);

}  // namespace res
