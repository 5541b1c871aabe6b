// Device building blocks of the streaming kernels (forward and backward):
// address-space views for direct-to-LDS loads, the time-major LDS tile of the
// forward, the 16x16 MFMA operand paths, complex steps across a lane pair, and
// explicit memory-counter waits.
#pragma once

#include "common.h"

namespace res {

typedef __attribute__((address_space(1))) void gvoid_t;
typedef __attribute__((address_space(3))) void lvoid_t;

// Time-major LDS tile of elements of ES bytes: rows of 128 bytes (the tile's
// channels), groups of 8 rows padded so that every group starts on a 16-byte
// boundary for the direct-to-LDS loads and row stores (bf16: +8 bytes, so the
// 8-byte operand gathers of 16 lanes from 16 different groups spread over the
// banks; float: +16 bytes).
constexpr int XROW = 128;
template <int ES> struct XLay {
  static constexpr int GRP = 8 * XROW + (ES == 2 ? 8 : 16);
  static constexpr int BYTES = (TILE_T / 8) * GRP;
  __device__ static __forceinline__ int off(int t) { return (t >> 3) * GRP + (t & 7) * XROW; }
};

// Time-major LDS tile of the single-pass forward: 256 rows of 128 bytes in eight
// 16-byte pieces, piece k of a row of chunk n (16 rows) in slot k ^ (n & 7), and
// for 2-byte elements the rows of chunks 8 .. 15 shifted by 8 bytes.  The operand
// reads and output writes of 16 lanes (one row of each chunk, 4 channels) then
// fall on different banks (8 bytes a lane over 16 chunks for bf16, 16 bytes over
// 8 chunks for float), and a group of 8 rows stays one contiguous kilobyte for
// the direct-to-LDS loads and row stores.
template <int ES> struct XTile {
  static constexpr int BYTES = TILE_T * XROW + 16;
  // byte offset of row group g (rows 8g .. 8g+7)
  __device__ static __forceinline__ int group(int g) { return g * (8 * XROW) + (ES == 2 ? (g >> 4) * 8 : 0); }
  // byte offset of channel byte cb (0 .. 127) of row t
  __device__ static __forceinline__ int off(int t, int cb) {
    return t * XROW + (ES == 2 ? (t >> 7) * 8 : 0) + ((((cb >> 4) ^ (t >> 4)) & 7) << 4) + (cb & 15);
  }
};

// Compiler-level ordering of LDS accesses inside one wave (the LDS executes a
// wave's accesses in program order).
__device__ __forceinline__ void wave_lds_order() { asm volatile("" ::: "memory"); }

// ---------------------------------------------------------------------------
// Forward operands: every product contracts one chunk (16 steps).
//   FPath<float>: four v_mfma_f32_16x16x4_f32, slot (kk, q) = index 4q + kk:
//     lane (i, q) holds A[i][4q..4q+3], lane (n, q) holds B[4q..4q+3][n].
//   FPath<bf16_t>: split-bf16 on v_mfma_f32_16x16x16_bf16.  A per-channel
//     matrix A (from float64) is stored as Ah = bf16(A), Al = bf16(A - Ah); lane
//     (i, q) holds Ah[i][4q..4q+3] then Al[i][4q..4q+3] (16 bytes).  The
//     activations are exact in bf16; lane (n, q) holds x[16n+4q .. 16n+4q+3],
//     and two instructions give (Ah + Al) x (tables at ~2^-17 relative).
// In both, lane (n, q) of the activation operand reads tile rows 16n + 4q + r,
// r = 0..3: group 2n + (q >> 1), rows 4 (q & 1) + r.
// ---------------------------------------------------------------------------
template <typename TX> struct FPath;
template <> struct FPath<float> {
  typedef f4 AOp;
  typedef f4 XOp;
  __device__ static __forceinline__ AOp load_a(const void* p) { return load_f4(p); }
  __device__ static __forceinline__ AOp load_a_u4(uint4 u) {
    const f4 r = {__uint_as_float(u.x), __uint_as_float(u.y), __uint_as_float(u.z), __uint_as_float(u.w)};
    return r;
  }
  // the operand of a lane's four float32 entries with all their bits
  typedef AOp AFull;
  __device__ static __forceinline__ AFull full_a(const float (&v)[4]) { return f4{v[0], v[1], v[2], v[3]}; }
  __device__ static __forceinline__ f4 mma(const AOp& a, const XOp& x, f4 c) { return mma_f32(a, x, c); }
  // (A x)^T: lane (i, q) gets columns 4q .. 4q+3 of row i of A x
  __device__ static __forceinline__ f4 mma_t(const XOp& x, const AOp& a, f4 c) { return mma_f32(x, a, c); }
  // y += U H for float32 states H (lane (n, q): components 4q .. 4q+3 of chunk n)
  typedef f4 UOp;
  __device__ static __forceinline__ UOp u_op(const f4& u) { return u; }
  __device__ static __forceinline__ f4 mma_u(const UOp& u, const f4& h, f4 c) { return mma_f32(u, h, c); }
  // y = T x + U H
  struct OOp {
    f4 t, u;
  };
  __device__ static __forceinline__ OOp o_op(const AOp& t, const f4& u) { return OOp{t, u}; }
  __device__ static __forceinline__ f4 out(const OOp& o, const XOp& x, const f4& h) {
    const f4 zero = {0.f, 0.f, 0.f, 0.f};
    return mma_f32(o.u, h, mma_f32(o.t, x, zero));
  }
  // the same from the byte address p of row 16n + 4q of an XTile
  __device__ static __forceinline__ void gather_rows(const char* p, XOp (&xv)[4]) {
#pragma unroll
    for (int kk = 0; kk < 4; ++kk) {
      const f4 w = *reinterpret_cast<const f4*>(p + kk * XROW);
#pragma unroll
      for (int c = 0; c < 4; ++c) xv[c][kk] = w[c];
    }
  }
  // the 4 consecutive channels ch0 .. ch0+3 (ch0 a multiple of 4), one 16-byte read per row
  __device__ static __forceinline__ void gather4(const char* xt, int ch0, int n, int q, XOp (&xv)[4]) {
    const char* p = xt + (2 * n + (q >> 1)) * XLay<4>::GRP + 4 * (q & 1) * XROW + ch0 * 4;
#pragma unroll
    for (int kk = 0; kk < 4; ++kk) {
      const f4 w = *reinterpret_cast<const f4*>(p + kk * XROW);
#pragma unroll
      for (int c = 0; c < 4; ++c) xv[c][kk] = w[c];
    }
  }
};
template <> struct FPath<bf16_t> {
  struct AOp {
    s4 hi, lo;
  };
  typedef s4 XOp;
  __device__ static __forceinline__ AOp load_a(const void* p) { return load_a_u4(*reinterpret_cast<const uint4*>(p)); }
  __device__ static __forceinline__ AOp load_a_u4(uint4 u) {
    AOp a;
    a.hi = __builtin_bit_cast(s4, make_uint2(u.x, u.y));
    a.lo = __builtin_bit_cast(s4, make_uint2(u.z, u.w));
    return a;
  }
  // the operand of a lane's four float32 entries with all their bits, in three
  // bf16 parts of 8 bits each (remainders as in split_h)
  struct AFull {
    s4 hi, mid, lo;
  };
  __device__ static __forceinline__ AFull full_a(const float (&v)[4]) {
    typedef __bf16 b2 __attribute__((ext_vector_type(2)));
    uint32_t u10 = 0x0000BF80u, u01 = 0xBF800000u;
    asm("" : "+s"(u10), "+s"(u01));
    const b2 m10 = __builtin_bit_cast(b2, u10), m01 = __builtin_bit_cast(b2, u01);
    uint32_t part[3][2];
#pragma unroll
    for (int i = 0; i < 2; ++i) {
      float r0 = v[2 * i], r1 = v[2 * i + 1];
#pragma unroll
      for (int j = 0; j < 3; ++j) {
        const b2 h = {(__bf16)r0, (__bf16)r1};
        part[j][i] = __builtin_bit_cast(uint32_t, h);
        if (j < 2) {
          r0 = __builtin_amdgcn_fdot2_f32_bf16(h, m10, r0, false);
          r1 = __builtin_amdgcn_fdot2_f32_bf16(h, m01, r1, false);
        }
      }
    }
    return AFull{__builtin_bit_cast(s4, make_uint2(part[0][0], part[0][1])),
                 __builtin_bit_cast(s4, make_uint2(part[1][0], part[1][1])),
                 __builtin_bit_cast(s4, make_uint2(part[2][0], part[2][1]))};
  }
  __device__ static __forceinline__ f4 mma(const AOp& a, const XOp& x, f4 c) {
    c = __builtin_amdgcn_mfma_f32_16x16x16bf16_1k(a.hi, x, c, 0, 0, 0);
    return __builtin_amdgcn_mfma_f32_16x16x16bf16_1k(a.lo, x, c, 0, 0, 0);
  }
  // (A x)^T: lane (i, q) gets columns 4q .. 4q+3 of row i of A x
  __device__ static __forceinline__ f4 mma_t(const XOp& x, const AOp& a, f4 c) {
    c = __builtin_amdgcn_mfma_f32_16x16x16bf16_1k(x, a.hi, c, 0, 0, 0);
    return __builtin_amdgcn_mfma_f32_16x16x16bf16_1k(x, a.lo, c, 0, 0, 0);
  }
  __device__ static __forceinline__ f4 mma_t(const XOp& x, const AFull& a, f4 c) {
    c = __builtin_amdgcn_mfma_f32_16x16x16bf16_1k(x, a.hi, c, 0, 0, 0);
    c = __builtin_amdgcn_mfma_f32_16x16x16bf16_1k(x, a.mid, c, 0, 0, 0);
    return __builtin_amdgcn_mfma_f32_16x16x16bf16_1k(x, a.lo, c, 0, 0, 0);
  }
  // y += U H for float32 states H (lane (n, q): components 4q .. 4q+3 of chunk n):
  // U (float32 table) and H split into bf16 halves, Uh Hh + Ul Hh + Uh Hl
  // (the omitted Ul Hl is ~2^-16 relative)
  typedef AOp UOp;
  __device__ static __forceinline__ UOp u_op(const f4& u) {
    UOp r;
    typedef __bf16 b4 __attribute__((ext_vector_type(4)));
    b4 hi, lo;
#pragma unroll
    for (int i = 0; i < 4; ++i) {
      hi[i] = (__bf16)u[i];
      lo[i] = (__bf16)(u[i] - (float)hi[i]);
    }
    r.hi = __builtin_bit_cast(s4, hi);
    r.lo = __builtin_bit_cast(s4, lo);
    return r;
  }
  // float32 states split into bf16 halves: pairs rounded together; each remainder
  // h - bf16(h) (exact: the two are within a factor of two) as one bf16 dot
  // product of the rounded pair with (-1, 0) or (0, -1), accumulated onto h
  __device__ static __forceinline__ void split_h(const f4& h, uint32_t (&ph)[2], uint32_t (&pl)[2]) {
    typedef __bf16 b2 __attribute__((ext_vector_type(2)));
    // the two selectors live in registers: a packed bf16 operand given as a
    // 32-bit inline constant is not read as the pair written here
    uint32_t u10 = 0x0000BF80u, u01 = 0xBF800000u;
    asm("" : "+s"(u10), "+s"(u01));
    const b2 m10 = __builtin_bit_cast(b2, u10), m01 = __builtin_bit_cast(b2, u01);
#pragma unroll
    for (int i = 0; i < 2; ++i) {
      const b2 hi = {(__bf16)h[2 * i], (__bf16)h[2 * i + 1]};
      ph[i] = __builtin_bit_cast(uint32_t, hi);
      const b2 lo = {(__bf16)__builtin_amdgcn_fdot2_f32_bf16(hi, m10, h[2 * i], false),
                     (__bf16)__builtin_amdgcn_fdot2_f32_bf16(hi, m01, h[2 * i + 1], false)};
      pl[i] = __builtin_bit_cast(uint32_t, lo);
    }
  }
  __device__ static __forceinline__ f4 mma_u(const UOp& u, const f4& h, f4 c) {
    uint32_t ph[2], pl[2];
    split_h(h, ph, pl);
    const s4 bh = __builtin_bit_cast(s4, make_uint2(ph[0], ph[1]));
    const s4 bl = __builtin_bit_cast(s4, make_uint2(pl[0], pl[1]));
    c = __builtin_amdgcn_mfma_f32_16x16x16bf16_1k(u.hi, bh, c, 0, 0, 0);
    c = __builtin_amdgcn_mfma_f32_16x16x16bf16_1k(u.lo, bh, c, 0, 0, 0);
    return __builtin_amdgcn_mfma_f32_16x16x16bf16_1k(u.hi, bl, c, 0, 0, 0);
  }
  // y = T x + U H as three 32-deep products: the contraction index is shared out
  // so that lane (n, q) holds steps 4q .. 4q+3 of x and then components
  // 4q .. 4q+3 of H; [Th | Uh] and [Tl | Ul] meet [x | Hh], and [Th | Uh] meets
  // [0 | Hl].  (Not a 16-deep product for the last: see mfma_depth_change.)
  struct OOp {
    bf8 hi, lo;
  };
  __device__ static __forceinline__ OOp o_op(const AOp& t, const f4& u) {
    const UOp w = u_op(u);
    OOp o;
    const uint2 th = __builtin_bit_cast(uint2, t.hi), tl = __builtin_bit_cast(uint2, t.lo);
    const uint2 uh = __builtin_bit_cast(uint2, w.hi), ul = __builtin_bit_cast(uint2, w.lo);
    o.hi = __builtin_bit_cast(bf8, make_uint4(th.x, th.y, uh.x, uh.y));
    o.lo = __builtin_bit_cast(bf8, make_uint4(tl.x, tl.y, ul.x, ul.y));
    return o;
  }
  __device__ static __forceinline__ f4 out(const OOp& o, const XOp& x, const f4& h) {
    uint32_t ph[2], pl[2];
    split_h(h, ph, pl);
    const uint2 xx = __builtin_bit_cast(uint2, x);
    const bf8 b = __builtin_bit_cast(bf8, make_uint4(xx.x, xx.y, ph[0], ph[1]));
    const bf8 bl = __builtin_bit_cast(bf8, make_uint4(0u, 0u, pl[0], pl[1]));
    f4 c = {0.f, 0.f, 0.f, 0.f};
    c = __builtin_amdgcn_mfma_f32_16x16x32_bf16(o.hi, b, c, 0, 0, 0);
    c = __builtin_amdgcn_mfma_f32_16x16x32_bf16(o.lo, b, c, 0, 0, 0);
    return __builtin_amdgcn_mfma_f32_16x16x32_bf16(o.hi, bl, c, 0, 0, 0);
  }
  // the same from the byte address p of row 16n + 4q of an XTile
  __device__ static __forceinline__ void gather_rows(const char* p, XOp (&xv)[4]) {
    typedef unsigned short us4 __attribute__((ext_vector_type(4)));
    us4 w[4];
#pragma unroll
    for (int r = 0; r < 4; ++r) w[r] = *reinterpret_cast<const us4*>(p + r * XROW);
#pragma unroll
    for (int c = 0; c < 4; ++c) {
      const us4 v = {w[0][c], w[1][c], w[2][c], w[3][c]};
      xv[c] = __builtin_bit_cast(s4, v);
    }
  }
  // the 4 consecutive channels ch0 .. ch0+3 (ch0 a multiple of 4): element r of
  // channel c from row r (the compiler reads each row once and packs with byte
  // permutes)
  __device__ static __forceinline__ void gather4(const char* xt, int ch0, int n, int q, XOp (&xv)[4]) {
    const char* p = xt + (2 * n + (q >> 1)) * XLay<2>::GRP + 4 * (q & 1) * XROW + ch0 * 2;
    typedef unsigned short us4 __attribute__((ext_vector_type(4)));
#pragma unroll
    for (int c = 0; c < 4; ++c) {
      us4 v;
#pragma unroll
      for (int r = 0; r < 4; ++r) v[r] = *reinterpret_cast<const unsigned short*>(p + r * XROW + c * 2);
      xv[c] = __builtin_bit_cast(s4, v);
    }
  }
};

__device__ __forceinline__ float swap_pair(float v) {  // value of the neighbouring lane (lane ^ 1)
  return __builtin_bit_cast(float, __builtin_amdgcn_update_dpp(0, __builtin_bit_cast(int, v), 0xB1,
                                                               0xF, 0xF, false));
}

// One complex multiply-add on the lane's component of a (re, im) lane pair:
// zr v + zs v' + add, with v' the value of lane i ^ 1 (the other component),
// zs = -Im z on the re lane and +Im z on the im lane.  The partner product is
// one fused multiply-add whose first operand is read across the pair (DPP
// quad_perm [1,0,3,2]).  A DPP read needs two wait states after a vector
// write of its source: the multiply-add on v, which must come between any
// write of v and this instruction, is one, the s_nop the other.
__device__ __forceinline__ float cfma_pair(float zr, float zs, float v, float add) {
  float acc = fmaf(zr, v, add);
  asm("s_nop 0\n\tv_fmac_f32_dpp %0, %1, %2 quad_perm:[1,0,3,2] row_mask:0xf bank_mask:0xf"
      : "+v"(acc)
      : "v"(v), "v"(zs));
  return acc;
}

// One 16-byte-per-lane load straight into LDS (64 lanes, 1 KB at lds) from
// base + off (base wave-uniform, off the lane's byte offset).  Issued as an
// opaque instruction: the compiler then does not wait for it before every later
// LDS read of the issuing wave (it cannot tell which buffer a read touches); the
// kernel waits for its own tiles explicitly (vmcnt) before the barrier that
// publishes them.
__device__ __forceinline__ void lds_dma16(const void* base, uint32_t off, const void* lds) {
  const uint32_t la = (uint32_t)(size_t)(lvoid_t*)lds;
  asm volatile("s_nop 0\n\tglobal_load_lds_dwordx4 %0, %1" ::"v"(off), "s"(base), "{m0}"(la) : "memory");
}

// The same from a 64-bit address per lane.
__device__ __forceinline__ void lds_dma16_lane(const void* src, const void* lds) {
  const uint32_t la = (uint32_t)(size_t)(lvoid_t*)lds;
  asm volatile("s_nop 0\n\tglobal_load_lds_dwordx4 %0, off" ::"v"((uint64_t)src), "{m0}"(la) : "memory");
}

// Wait until at most N vector memory operations of the wave are outstanding.
template <int N>
__device__ __forceinline__ void wait_vm() {
  static_assert(N >= 0 && N < 64, "a six-bit count");
  __builtin_amdgcn_s_waitcnt(0x0F70 | (N & 15) | ((N >> 4) << 14));
}

// Wait until at most n (0 <= n <= 63) vector memory operations of the wave are
// outstanding (exp and lgkm counts not waited for).
__device__ __forceinline__ void wait_vmcnt(int n) {
  switch (n) {
#define RES_VMC(k) \
  case k: __builtin_amdgcn_s_waitcnt(0x0F70 | ((k) & 15) | (((k) >> 4) << 14)); break;
#define RES_VMC8(k) RES_VMC(k) RES_VMC(k + 1) RES_VMC(k + 2) RES_VMC(k + 3) RES_VMC(k + 4) RES_VMC(k + 5) \
  RES_VMC(k + 6) RES_VMC(k + 7)
    RES_VMC8(0) RES_VMC8(8) RES_VMC8(16) RES_VMC8(24) RES_VMC8(32) RES_VMC8(40) RES_VMC8(48) RES_VMC8(56)
#undef RES_VMC8
#undef RES_VMC
    default: __builtin_amdgcn_s_waitcnt(0x0F70); break;
  }
}

// 16-byte store of each lane to base + off (base wave-uniform), as an opaque
// instruction like lds_dma16, so that the compiler keeps the 64-bit base in
// scalar registers and the lane offset in one vector register.  A store of more
// than 8 bytes reads its data registers after issue: on gfx950 a vector write to
// them needs two wait states after the store, which the compiler's hazard
// tracking cannot see inside an asm statement, so the asm carries them.  The
// rows are outputs no work-group reads again, so the store is non-temporal
// (nt): it does not leave dirty lines in the L2 to be written back when the
// kernel ends (the forward at B4 L32K bf16: 65 to 60 us a launch).
typedef uint32_t u32x4 __attribute__((ext_vector_type(4)));
__device__ __forceinline__ void st_row16(void* base, uint32_t off, u32x4 v) {
  asm volatile("global_store_dwordx4 %0, %1, %2 nt\n\ts_nop 1" ::"v"(off), "v"(v), "s"(base) : "memory");
}

// Transposition of the chunk sums of 4 channels across the wave: R[k] holds
// channel k with lane (i, q) carrying component i of chunks 4q .. 4q+3 (the
// transposed product layout); afterwards lane (i, c) holds component i of
// chunks 0 .. 15 of channel c in S[0 .. 15] (permlane swaps of 32 and 16 lanes).
__device__ __forceinline__ void lanes_to_chunks(const f4 (&R)[4], float (&S)[16]) {
#pragma unroll
  for (int r = 0; r < 4; ++r) {
    const uint32_t v0 = __float_as_uint(R[0][r]), v1 = __float_as_uint(R[1][r]);
    const uint32_t v2 = __float_as_uint(R[2][r]), v3 = __float_as_uint(R[3][r]);
    const auto s02 = __builtin_amdgcn_permlane32_swap(v0, v2, false, false);
    const auto s13 = __builtin_amdgcn_permlane32_swap(v1, v3, false, false);
    const auto s01 = __builtin_amdgcn_permlane16_swap(s02[0], s13[0], false, false);
    const auto s23 = __builtin_amdgcn_permlane16_swap(s02[1], s13[1], false, false);
    S[r] = __uint_as_float(s01[0]);
    S[4 + r] = __uint_as_float(s01[1]);
    S[8 + r] = __uint_as_float(s23[0]);
    S[12 + r] = __uint_as_float(s23[1]);
  }
}

}  // namespace res
