// Device code shared by the kernels that quantize Q, K and V (sage_prologue.hip, sage_attn_raw.hip): loads, the quantizer
// psi of Sec. 2.2 and the packing of its codes.
#pragma once
#include "sage_common.h"

namespace sage {

// 16-byte load marked non-temporal: Q, K and V are streamed once per pass, and keeping them out of the
// way of the caches measured 25 % faster on the statistics pass
__device__ inline uint4 nt_load16(const unsigned short* p) {
  typedef unsigned v4u __attribute__((ext_vector_type(4)));
  const v4u r = __builtin_nontemporal_load(reinterpret_cast<const v4u*>(p));
  return make_uint4(r[0], r[1], r[2], r[3]);
}

__device__ inline uint2 nt_load8(const unsigned short* p) {
  typedef unsigned v2u __attribute__((ext_vector_type(2)));
  const v2u r = __builtin_nontemporal_load(reinterpret_cast<const v2u*>(p));
  return make_uint2(r[0], r[1]);
}

template <bool BF16, bool NT = true>
__device__ inline void load8(const unsigned short* p, float (&x)[8]) {
  const uint4 raw = NT ? nt_load16(p) : *reinterpret_cast<const uint4*>(p);
  const unsigned w[4] = {raw.x, raw.y, raw.z, raw.w};
#pragma unroll
  for (int i = 0; i < 4; ++i) {
    x[2 * i] = load16<BF16>((unsigned short)(w[i] & 0xffffu));
    x[2 * i + 1] = load16<BF16>((unsigned short)(w[i] >> 16));
  }
}

template <bool BF16>
__device__ inline void unpack8(const uint4& raw, float* x) {
  const unsigned w[4] = {raw.x, raw.y, raw.z, raw.w};
#pragma unroll
  for (int i = 0; i < 4; ++i) {
    x[2 * i] = load16<BF16>((unsigned short)(w[i] & 0xffffu));
    x[2 * i + 1] = load16<BF16>((unsigned short)(w[i] >> 16));
  }
}

// The value of lane l ^ O - one step of a butterfly - without an LDS round trip: data-parallel moves inside 16 lanes (steps
// of 16 and 32 exchange register halves instead, below).  For O = 4 the move mirrors half a row, which is lane l ^ 4 where the
// lanes of a quad agree: that step comes after 1 and 2.
template <int O>
__device__ __forceinline__ unsigned butterfly(unsigned u) {
  static_assert(O == 1 || O == 2 || O == 4 || O == 8, "a step inside 16 lanes");
  constexpr int CTRL = O == 1 ? 0xB1 : (O == 2 ? 0x4E : (O == 4 ? 0x141 : 0x128));   // quad_perm, row_half_mirror, row_ror:8
  return (unsigned)__builtin_amdgcn_update_dpp(0, (int)u, CTRL, 0xf, 0xf, true);
}
template <int O> __device__ __forceinline__ float butterfly_max(float v) {
  if constexpr (O == 16 || O == 32) {
    const unsigned u = __float_as_uint(v);
    const auto r = O == 16 ? __builtin_amdgcn_permlane16_swap(u, u, false, false) : __builtin_amdgcn_permlane32_swap(u, u, false, false);
    return fmaxf(__uint_as_float(r[0]), __uint_as_float(r[1]));
  } else {
    return fmaxf(v, __uint_as_float(butterfly<O>(__float_as_uint(v))));
  }
}
template <int O> __device__ __forceinline__ double butterfly_sum(double v) {
  const unsigned long long b = __double_as_longlong(v);
  const unsigned lo = (unsigned)b, hi = (unsigned)(b >> 32);
  auto join = [](unsigned l, unsigned h) { return __longlong_as_double((long long)(((unsigned long long)h << 32) | l)); };
  if constexpr (O == 16 || O == 32) {
    const auto rl = O == 16 ? __builtin_amdgcn_permlane16_swap(lo, lo, false, false) : __builtin_amdgcn_permlane32_swap(lo, lo, false, false);
    const auto rh = O == 16 ? __builtin_amdgcn_permlane16_swap(hi, hi, false, false) : __builtin_amdgcn_permlane32_swap(hi, hi, false, false);
    return join(rl[0], rh[0]) + join(rl[1], rh[1]);
  } else {
    return v + join(butterfly<O>(lo), butterfly<O>(hi));
  }
}
// over groups of N consecutive lanes
template <int N> __device__ __forceinline__ float group_max(float v) {
  v = butterfly_max<1>(v);
  if constexpr (N > 2) v = butterfly_max<2>(v);
  if constexpr (N > 4) v = butterfly_max<4>(v);
  if constexpr (N > 8) v = butterfly_max<8>(v);
  if constexpr (N > 16) v = butterfly_max<16>(v);
  if constexpr (N > 32) v = butterfly_max<32>(v);
  return v;
}
__device__ __forceinline__ float wave_max(float v) { return group_max<64>(v); }

// x / s rounded to nearest, given r = fl32(1 / s): the quotient corrected by its exact remainder (Markstein), three
// instructions.  Correct for every s that div_by_ok accepts (the mantissa of all ones is the theorem's exception), except
// where the remainder underflows: quotients below 2^-40, which every 8-bit and 4-bit code rounds to 0.
__device__ __forceinline__ float div_by(float x, float s, float r) {
  const float q = __fmul_rn(x, r);
  return __fmaf_rn(__fmaf_rn(q, -s, x), r, q);
}
__device__ __forceinline__ bool div_by_ok(float s) {
  return s >= 0x1p-60f && s <= 0x1p60f && (__float_as_uint(s) & 0x7fffffu) != 0x7fffffu;
}

// psi of Sec. 2.2: code = clip(round-half-even(x / delta)); delta == 0 gives code 0.
__device__ inline int quant_code(float x, float delta, int qmax) {
  if (!(delta > 0.0f)) return 0;
  const float r = rintf(__fdiv_rn(x, delta));
  const int c = (int)r;
  return c > qmax ? qmax : (c < -qmax ? -qmax : c);
}

// psi with the correctly rounded quotient of div_by, for whole wavefronts: `fast` says that every lane's scale is one that
// div_by accepts, or zero (all its values are then zero and so are their codes).  Three multiply-adds and a rounding per code and no
// branch per eight codes (a product with the reciprocal whose distance from the next half-integer was watched, and a division where it was too
// near, took a difference and a maximum more).
struct CodeScale { float r; bool fast; };
__device__ __forceinline__ CodeScale code_scale(float delta) {
  CodeScale q;
  q.fast = __builtin_amdgcn_ballot_w64(!(div_by_ok(delta) || delta == 0.0f)) == 0;
  q.r = q.fast && delta > 0.0f ? __fdiv_rn(1.0f, delta) : 0.0f;
  return q;
}
// NE codes as integer-valued floats, handed to put(e, code)
template <int NE, int QMAX, class Put>
__device__ __forceinline__ void code_group(const float* x, float delta, const CodeScale& qs, Put&& put) {
  if (qs.fast) {
#pragma unroll
    for (int e = 0; e < NE; ++e) put(e, rintf(div_by(x[e], delta, qs.r)));
  } else {
#pragma unroll
    for (int e = 0; e < NE; ++e) {
      float c = (float)quant_code(x[e], delta, QMAX);
      asm volatile("" : "+v"(c) :: "memory");          // (one division at a time: together they want more registers than the loop has)
      put(e, c);
    }
  }
}
// ... in the low bytes of c[0..NE) (adding 1.5 * 2^23 rounds to the nearest integer, ties to even, and leaves it in the low
// mantissa bits)
template <int NE, int QMAX>
__device__ __forceinline__ void code_group_bytes(const float* x, float delta, const CodeScale& qs, unsigned (&c)[NE]) {
  if (qs.fast) {
#pragma unroll
    for (int e = 0; e < NE; ++e) c[e] = __float_as_uint(div_by(x[e], delta, qs.r) + 12582912.0f);
  } else {
#pragma unroll
    for (int e = 0; e < NE; ++e) {
      c[e] = (unsigned)quant_code(x[e], delta, QMAX);
      asm volatile("" : "+v"(c[e]) :: "memory");
    }
  }
}
// the low bytes of four words side by side
__device__ __forceinline__ unsigned pack4(const unsigned* c) {
  return __builtin_amdgcn_perm(__builtin_amdgcn_perm(c[3], c[2], 0x0c0c0400u), __builtin_amdgcn_perm(c[1], c[0], 0x0c0c0400u), 0x05040100u);
}
// ... of sixteen
__device__ __forceinline__ uint4 pack16(const unsigned (&c)[16]) { return make_uint4(pack4(c), pack4(c + 4), pack4(c + 8), pack4(c + 12)); }

typedef unsigned v6u __attribute__((ext_vector_type(6)));
// 32 INT4 codes held as integer-valued floats (every integer of [-7, 7] is an E2M3 value) become
// consecutive 6-bit E2M3 fields, element e at bit 6e: the conversion instruction takes the even
// elements in its first operand and the odd ones in its second (scale 1.0), so the codes are
// collected in that shape from the start
struct Codes32 {
  v16f ev, od;
  __device__ inline void set(int e, float c) { if (e & 1) od[e >> 1] = c; else ev[e >> 1] = c; }
  // The instruction writes its first result registers before it has read all of its inputs, and
  // the compiler does not know: a result allocated on top of part of an input corrupts the codes.
  // The empty asm statements make both operands opaque 16-register values and then need them and
  // the result at the same time, which keeps the three register ranges apart.  (Vector operands
  // of asm statements do not parse in the host pass, which never calls this.)
  __device__ inline v6u pack() const {
    v6u r = {0u, 0u, 0u, 0u, 0u, 0u};
#if defined(__HIP_DEVICE_COMPILE__)
    v16f a = ev, b = od;
    asm volatile("" : "+v"(a), "+v"(b));
    r = __builtin_amdgcn_cvt_scalef32_2xpk16_fp6_f32(a, b, 1.0f);
    asm volatile("" ::"v"(r), "v"(a), "v"(b));
#endif
    return r;
  }
};

// A row of 256 16-bit values by four lanes l, l + 16, l + 32, l + 48 (kk = 0..3), each of which wants 64 consecutive values
// (pieces 8 kk .. of 8 values).  Loaded that way, a load instruction touches 16 bytes of a lane's 128, and the eight
// instructions meet in the caches or not at all.  Instead instruction i loads piece quad_piece(i, kk) - the
// four lanes side by side, 64 bytes - and quad_exchange moves the pieces to their lanes, in registers.
// In bits: the pieces' number is (i, kk) with the low two bits in the lane; exchanging a register bit with a lane bit is
// one v_permlane32_swap or v_permlane16_swap per pair of registers.  (Rows of 64 and 128 values, where a lane's piece is a part
// of one cache line, are faster without.)
__device__ __forceinline__ int quad_piece(int i, int kk) { return 4 * i + kk; }
__device__ __forceinline__ void quad_swap32(uint4& a, uint4& b) {
  auto r = __builtin_amdgcn_permlane32_swap(a.x, b.x, false, false); a.x = r[0]; b.x = r[1];
  r = __builtin_amdgcn_permlane32_swap(a.y, b.y, false, false); a.y = r[0]; b.y = r[1];
  r = __builtin_amdgcn_permlane32_swap(a.z, b.z, false, false); a.z = r[0]; b.z = r[1];
  r = __builtin_amdgcn_permlane32_swap(a.w, b.w, false, false); a.w = r[0]; b.w = r[1];
}
__device__ __forceinline__ void quad_swap16(uint4& a, uint4& b) {
  auto r = __builtin_amdgcn_permlane16_swap(a.x, b.x, false, false); a.x = r[0]; b.x = r[1];
  r = __builtin_amdgcn_permlane16_swap(a.y, b.y, false, false); a.y = r[0]; b.y = r[1];
  r = __builtin_amdgcn_permlane16_swap(a.z, b.z, false, false); a.z = r[0]; b.z = r[1];
  r = __builtin_amdgcn_permlane16_swap(a.w, b.w, false, false); a.w = r[0]; b.w = r[1];
}
__device__ __forceinline__ void quad_exchange(uint4 (&x)[8]) {     // (p4 p3 p2; p1 p0) -> (p1 p0 p2; p4 p3), then the registers in order
  quad_swap32(x[0], x[4]); quad_swap32(x[1], x[5]); quad_swap32(x[2], x[6]); quad_swap32(x[3], x[7]);
  quad_swap16(x[0], x[2]); quad_swap16(x[1], x[3]); quad_swap16(x[4], x[6]); quad_swap16(x[5], x[7]);
  const uint4 y[8] = {x[0], x[2], x[4], x[6], x[1], x[3], x[5], x[7]};
#pragma unroll
  for (int i = 0; i < 8; ++i) x[i] = y[i];
}

}  // namespace sage
