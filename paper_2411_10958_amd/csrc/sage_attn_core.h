// Device code shared by the attention kernels (sage_attn_kernel.hip, sage_attn_raw.hip): their arguments, the score
// product, the softmax pieces and the P~V product of Algorithm 1's inner loop for one wavefront.
#pragma once
#include "sage_common.h"

namespace sage {

struct AttnParams {
  const int8_t* q_codes;
  const int8_t* k_codes;
  const uint8_t* v_codes;
  const float* q_scale;
  const float* k_scale;
  const float* v_scale;
  const float* v_mean;    // null, or the token mean of V to add back (smooth-V option)
  const float* delta_s;
  void* out;
  int H, Hkv, N, Nk, nQb, nKb, total_tiles;   // N queries, Nk keys (of the longest sequence)
  TensorMap om;           // where the rows of `out` start
  float kappa;
  SeqMap seq;             // variable-length batch: N, Nk, nQb, nKb describe the longest sequence
  float* lse;             // null, or where the row log-sum-exp goes
  const float* q_corr;    // kappa * <q_r, mean(K)> per query (read only with lse)
  int B;
  // key range split over several workgroups per tile (few tiles, many keys): partial results, merged by k_merge_splits
  int splits;             // workgroups per tile (1: no split)
  float* part_o;          // [tile * splits + s][128 rows][d]: unnormalized O under the chunk's own exponent offset
  float* part_el;         // [tile * splits + s][128 rows][2]: that offset e and the sum l under it
};

inline AttnParams attn_params(const Dims& Dm, const Ptrs& P) {
  AttnParams p;
  p.q_codes = P.q_codes; p.k_codes = P.k_codes; p.v_codes = P.v_codes;
  p.q_scale = P.q_scale; p.k_scale = P.k_scale; p.v_scale = P.v_scale; p.delta_s = P.delta_s;
  p.v_mean = Dm.smooth_v ? P.v_mean : nullptr;
  p.out = P.out;
  p.H = Dm.H; p.Hkv = Dm.Hkv; p.N = Dm.N; p.Nk = Dm.Nk; p.nQb = Dm.nQb; p.nKb = Dm.nKb;
  p.om = make_tensor_map(Dm.nhd, Dm.H, Dm.N, Dm.d, Dm.seq.cu_q != nullptr);
  p.seq = Dm.seq;
  p.lse = P.lse; p.q_corr = P.q_corr; p.B = Dm.B;
  p.total_tiles = Dm.B * Dm.H * Dm.nQb;
  p.kappa = Dm.kappa;
  p.splits = Dm.splits; p.part_o = P.part_o; p.part_el = P.part_el;
  return p;
}
// merge of the chunks of packed tiles (p.total_tiles of them: one per batch and KV head)
hipError_t launch_merge_packed(const Dims& Dm, const AttnParams& p, hipStream_t s);

// Whether the tiles of a packed batch of B sequences of at most N queries, `tokens` in all, go out in bands (in k_attn_fwd) or in the order
// of a fixed-length batch.  What the bands mend is raggedness, so the rule asks for it: a batch of (nearly) equal sequences has the
// heavy tiles of all of them first in the old order too, and its groups of heads share more.  Attention alone, us, old order / bands.
// No mask, by the part of B N that is there: 1 (41 of 500, 32 heads) 155 / 161, (8 of 8192, 32 heads) 5088 / 5459, 0.96 (16 of
// 2000, 64 channels) 239 / 246, 0.94 (8 of 4096, 32 heads) 1301 / 1268, 0.88 1266 / 1169, 0.75 1238 / 931, 0.36 1127 / 433; (31 of
// 6000) 0.19 2710 / 928; over 116 batches bands take 0.81 of the time, with the line at 0.9 or at 1 too, the worst under it 1.15 (64 of
// up to 662, 2 heads of 256 channels).  Causal: 1 (8 of 4096, 8 heads of 256 channels) 297 / 314, (12 of 2000) 132 / 144, (8 of 8192, 32
// heads) 2735 / 2807, 0.90 (16 of 2000) 155 / 161, 0.75 (8 of 4096, 16 heads of 64 channels) 167 / 172, 0.62 (16 of 2000, 8 heads of 256
// channels) 144 / 102, 0.36 (8 of 4096, 32 heads) 223 / 206, 0.29 (61 of 2500, 32 heads) 399 / 374, 0.19 (31 of 6000, 16 heads) 258 / 238, but with 32 heads 445 / 462; over 188
// batches of 600 to 40000 tiles 0.96, the worst under the line 1.08.  One band is no order: causal batches of up to BAND_LEVELS positions
// lose (41 of 500, 8 heads of 256 channels 59 / 68, 32 of up to 407 17.8 / 20.7).
constexpr int BAND_LEVELS = 4;
__host__ __device__ inline bool packed_in_bands(bool causal, int tokens, int B, int N) {
  const long long full = (long long)B * N;
  return causal ? N > BAND_LEVELS * BQ && 16LL * tokens < 13 * full : 32LL * tokens < 31 * full;
}

// Split of a tile's key blocks [0, nblk) into chunks, one workgroup each (Sec. 2.1, Eq. 1: the running maximum / sum /
// output of disjoint key sets combine by the same rule that combines consecutive blocks).  Every chunk must start
// with a block in which every query of the tile sees a key, so the chunks divide the first n_vis blocks - those
// with a key visible to the tile's first query - evenly, C = ceil(n_vis / S) blocks each, and the last non-empty
// chunk runs on to nblk; chunks s >= ceil(n_vis / C) are empty.
struct KeyChunk { int j0, j1; };
__host__ __device__ inline KeyChunk key_chunk(int s, int S, int nblk, int n_vis) {
  const int C = (n_vis + S - 1) / S;
  const int used = C > 0 ? (n_vis + C - 1) / C : 0;
  KeyChunk k;
  k.j0 = s * C;
  k.j1 = s + 1 >= used ? nblk : (s + 1) * C;
  if (s >= used) { k.j0 = k.j1 = 0; }
  return k;
}

// Score accumulators of one wavefront for one 64-key block: 2 key tiles x (32 keys x 32
// queries).  ka: the block's K^ chunks already in registers (chunk (s, kt) at ka[2s + kt]); qreg:
// the wavefront's Q^ B-operands (one per 32-channel step).  Element acc[kt][v] belongs to key
// 32*kt + 16*(lane/32) + v of the block and to query lane%32 of the wavefront.
// INT8 mode: v_mfma_i32_32x32x32_i8, int32 accumulators.  INT4 mode: the codes are 6-bit FP6 E2M3
// values and feed v_mfma_f32_32x32x64_f8f6f4 in its FP6 operand format (twice the rate of the 8-bit
// formats); the FP32 accumulators hold the exact integers.  Either way the result is returned as
// raw 32-bit lanes.
// The product is issued one MFMA ("step") at a time so that the steps can be spread between
// pieces of vector work: step I works on key tile I % 2 and contraction piece I / 2 (64 channels
// in the INT4 mode, 32 in the INT8 mode); the first piece of a tile starts from a zero accumulator.
// Operand registers: INT8 mode one 16-byte chunk per (piece, tile); INT4 mode one FP6 payload (24
// bytes in the low 6 dwords of an 8-dword operand) per (piece, tile).
template <bool INT4> struct QkOperand { typedef v4i type; };
template <> struct QkOperand<true> { typedef v8i type; };
template <bool INT4> using qk_operand_t = typename QkOperand<INT4>::type;
template <int D, bool INT4> constexpr int qk_pieces() { return INT4 ? D / 64 : D / 32; }
template <int D, bool INT4> constexpr int qk_steps() { return 2 * qk_pieces<D, INT4>(); }
template <int D, bool INT4> struct KBlockRegs { typedef qk_operand_t<INT4> type[2 * (INT4 ? D / 64 : D / 32)]; };

template <int D, bool INT4, int I>
__device__ __forceinline__ void qk_step(const typename QkOperand<INT4>::type (&ka)[qk_steps<D, INT4>()],
                                        const typename QkOperand<INT4>::type (&qreg)[qk_pieces<D, INT4>()],
                                        v16i (&acc)[2]) {
  constexpr int KT = I & 1, S = I >> 1;
  if constexpr (INT4) {
    v16f c;
#pragma unroll
    for (int v = 0; v < 16; ++v) c[v] = S == 0 ? 0.0f : __int_as_float(acc[KT][v]);
    // operand format 2 = FP6 E2M3 for both A and B
    c = __builtin_amdgcn_mfma_scale_f32_32x32x64_f8f6f4(ka[S * 2 + KT], qreg[S], c, 2, 2, 0, 0, 0, 0);
#pragma unroll
    for (int v = 0; v < 16; ++v) acc[KT][v] = __float_as_int(c[v]);
  } else {
    v16i c;
#pragma unroll
    for (int v = 0; v < 16; ++v) c[v] = S == 0 ? 0 : acc[KT][v];
    acc[KT] = __builtin_amdgcn_mfma_i32_32x32x32_i8(ka[S * 2 + KT], qreg[S], c, 0, 0, 0);
  }
}
template <int D, bool INT4, int I = 0>
__device__ __forceinline__ void qk_tile(const typename QkOperand<INT4>::type (&ka)[qk_steps<D, INT4>()],
                                        const typename QkOperand<INT4>::type (&qreg)[qk_pieces<D, INT4>()],
                                        v16i (&acc)[2]) {
  if constexpr (I < qk_steps<D, INT4>()) {
    qk_step<D, INT4, I>(ka, qreg, acc);
    qk_tile<D, INT4, I + 1>(ka, qreg, acc);
  }
}

// The steps of one key tile alone.
template <int D, bool INT4, int KT, int S = 0>
__device__ __forceinline__ void qk_key_tile(const typename QkOperand<INT4>::type (&ka)[qk_steps<D, INT4>()],
                                            const typename QkOperand<INT4>::type (&qreg)[qk_pieces<D, INT4>()],
                                            v16i (&acc)[2]) {
  if constexpr (S < qk_pieces<D, INT4>()) {
    qk_step<D, INT4, 2 * S + KT>(ka, qreg, acc);
    qk_key_tile<D, INT4, KT, S + 1>(ka, qreg, acc);
  }
}

// One (piece, tile) operand out of a packed K^ block or Q^ tile at `base` (LDS or global): INT8
// mode chunk `op`*64 + lane; INT4 mode the lane's 16 bytes of op's first plane and 8 bytes of its
// second plane.
template <bool INT4, typename Ptr>
__device__ __forceinline__ typename QkOperand<INT4>::type load_qk_operand(Ptr base, int op, int lane) {
  if constexpr (INT4) {
    const v4i lo = base[op * (OP6_BYTES / 16) + lane];
    const uint2 hi = *reinterpret_cast<const uint2*>(reinterpret_cast<const char*>(&base[op * (OP6_BYTES / 16) + 64]) + 8 * lane);
    v8i r;
    r[0] = lo[0]; r[1] = lo[1]; r[2] = lo[2]; r[3] = lo[3];
    r[4] = (int)hi.x; r[5] = (int)hi.y; r[6] = 0; r[7] = 0;
    return r;
  } else {
    return base[op * 64 + lane];
  }
}

// The K^ operands of one block out of LDS (blk: the block's packed image).
// INT4 mode: an operand is a 16-byte read plus an 8-byte read (its "tail").  Left free, the compiler pairs the
// tails of two operands into one two-address read and then moves the halves of its result next to their
// operands' first four registers, two vector instructions per operand in a loop that is bound by them.  The
// empty statement after every operand is a fence for memory accesses: reads cannot be merged across it, so
// every tail stays a read of its own that lands where its operand wants it, while the compiler still knows
// about every read and waits for it before the first use.
template <int D, bool INT4, typename Ptr>
__device__ __forceinline__ void read_k_block(Ptr blk, int lane, typename KBlockRegs<D, INT4>::type& ka) {
  constexpr int NS = qk_steps<D, INT4>();
#pragma unroll
  for (int i = 0; i < NS; ++i) {
    ka[i] = load_qk_operand<INT4>(blk, i, lane);
    if constexpr (INT4) asm volatile("" ::: "memory");
  }
}

// Per-wavefront running state of Algorithm 1's inner loop.
template <int D> struct RowState {
  v16f O[D / 32];   // cross-block FP32 accumulator; O[ct][v]: channel 32ct + 8(v/4) + 4(lane/32) + v%4
  float m_run;      // running max of the base-2 scores of this lane's query
  float l_run;      // this lane's share of the running sum of 448 * P~
};

// Quantization granularity of the keys as the kernel sees it (template parameter GM): a lane's 32
// scores of a block are (key tile KT, quad G, R) = key 32 KT + 16 (lane / 32) + 4 G + R, so
//   GM 0: one scale per run of 16 keys = one per key tile  (2 per lane and block; queries in pairs),
//   GM 1: one scale per run of 4 keys  = one per quad      (8 per lane and block; every query its own),
//   GM 2: one scale per key            = one per score     (32 per lane and block; every query its own).
// KeyScales: the block's key scales this lane needs; Factors: c = fl32(fl32(delta_Q delta_K) kappa).
template <int GM> struct KeyScales;
template <> struct KeyScales<0> { float s[2]; };
template <> struct KeyScales<1> { v4f s[2]; };
template <> struct KeyScales<2> { v4f s[2][4]; };
template <int GM> struct Factors;
template <> struct Factors<0> {
  float c[2];
  __device__ __forceinline__ void set(float dq, float kappa, const KeyScales<0>& k) {
    c[0] = __fmul_rn(__fmul_rn(dq, k.s[0]), kappa);
    c[1] = __fmul_rn(__fmul_rn(dq, k.s[1]), kappa);
  }
  __device__ __forceinline__ float at(int kt, int, int) const { return c[kt]; }
};
template <> struct Factors<1> {
  float c[2][4];
  __device__ __forceinline__ void set(float dq, float kappa, const KeyScales<1>& k) {
#pragma unroll
    for (int kt = 0; kt < 2; ++kt) {
#pragma unroll
      for (int g = 0; g < 4; ++g) c[kt][g] = __fmul_rn(__fmul_rn(dq, k.s[kt][g]), kappa);
    }
  }
  __device__ __forceinline__ float at(int kt, int g, int) const { return c[kt][g]; }
};
template <> struct Factors<2> {
  float c[2][4][4];
  __device__ __forceinline__ void set(float dq, float kappa, const KeyScales<2>& k) {
#pragma unroll
    for (int kt = 0; kt < 2; ++kt) {
#pragma unroll
      for (int g = 0; g < 4; ++g) {
#pragma unroll
        for (int r = 0; r < 4; ++r) c[kt][g][r] = __fmul_rn(__fmul_rn(dq, k.s[kt][g][r]), kappa);
      }
    }
  }
  __device__ __forceinline__ float at(int kt, int g, int r) const { return c[kt][g][r]; }
};
// The 8-bit mode has no Delta-S in its score line: the dequantization product is fused into the exponent's
// argument, 2^(fma(acc, c, -m)), one rounding, whatever the granularity of the key scales (with a scale per key
// nothing is saved - the maximum needs the products anyway - but the value that decides the FP8 code of P~ is
// formed the same way for every group map).
template <bool INT4, int GM> constexpr bool fused_factor() { return !INT4; }

// Middle part of one block of Algorithm 1's inner loop for one wavefront, cut into pieces of four
// keys (one "group": registers 4G..4G+3 of key tile KT) so that MFMAs can be issued between them.
//
// dequant_group: the raw scores of the group are dequantized (+ Delta-S) into sc, in base 2
// (Algorithm 1, score line); MASKED adds the causal diagonal (keys past last_visible) and the
// padded keys (n_keys and beyond).  In the INT8
// mode there is no Delta-S and one positive factor c per key tile, so sc keeps the accumulators
// as floats: the maximum commutes with the factor and the product is fused into the exponent's
// argument (exp_group), one instruction less per score.
template <bool INT4, bool CAUSAL, bool MASKED, int GM, int KT, int G>
__device__ __forceinline__ void dequant_group(const v16i (&raw)[2], v16i (&sc)[2], const Factors<GM>& fac, int half,
                                              int key0, int last_visible, int n_keys) {
#pragma unroll
  for (int r = 0; r < 4; ++r) {
    float x;
    if constexpr (INT4) {
      // On entry sc holds the block's Delta-S values (read from LDS straight into these registers): the score is
      // one fused multiply-add in place (the two-operand encoding, which issues faster than the three-operand
      // one).  Written as an ordinary expression, not as inline assembly: the compiler must see that it reads the
      // accumulators of a matrix instruction, or it cannot keep the wait states that read needs.
      x = __builtin_fmaf(__int_as_float(raw[KT][4 * G + r]), fac.at(KT, G, r), __int_as_float(sc[KT][4 * G + r]));
    }
    else x = (float)raw[KT][4 * G + r];       // 8-bit mode: the factor is applied inside the exponent's argument
    if constexpr (MASKED) {
      const int key = key0 + 32 * KT + 16 * half + 4 * G + r;
      if (key >= n_keys || (CAUSAL && key > last_visible)) x = -INFINITY;
    }
    sc[KT][4 * G + r] = __float_as_int(x);
  }
}

// update_max: running max over the block's 64 dequantized scores of this lane's query (Eq. 1 /
// Algorithm 1); takes the previous block's exponent offset in m_sub and returns the new one there, and
// alpha = 2^(old offset - new offset).
template <int D, bool INT4, int GM, int PVF>
__device__ __forceinline__ float update_max(RowState<D>& st, const v16i (&acc)[2], const Factors<GM>& fac,
                                            float& m_sub) {
  float mx;
  if constexpr (!fused_factor<INT4, GM>()) {
    mx = fmaxf(__int_as_float(acc[0][0]), __int_as_float(acc[1][0]));
#pragma unroll
    for (int v = 1; v < 16; ++v)   // one v_max3_f32 per step
      mx = fmaxf(fmaxf(mx, __int_as_float(acc[0][v])), __int_as_float(acc[1][v]));
  } else if constexpr (GM == 0) {
    // per key tile: max of the accumulators, then the tile's factor (c >= 0, so the order does not
    // matter; a fully masked tile with c = 0 gives NaN, which fmaxf drops)
    float m0 = __int_as_float(acc[0][0]), m1 = __int_as_float(acc[1][0]);
#pragma unroll
    for (int v = 1; v < 16; v += 2) {
      m0 = fmaxf(fmaxf(m0, __int_as_float(acc[0][v])), __int_as_float(acc[0][(v + 1) & 15]));
      m1 = fmaxf(fmaxf(m1, __int_as_float(acc[1][v])), __int_as_float(acc[1][(v + 1) & 15]));
    }
    // |c|: the pipeline's last update works on a stale, fully masked block whose scales are arbitrary
    // bits; -inf * |c| is -inf or NaN (dropped) whatever they are, so the running max stays intact
    mx = fmaxf(__fmul_rn(m0, fabsf(fac.at(0, 0, 0))), __fmul_rn(m1, fabsf(fac.at(1, 0, 0))));
  } else if constexpr (GM == 1) {
    // the same per quad
    mx = -INFINITY;
#pragma unroll
    for (int kt = 0; kt < 2; ++kt) {
#pragma unroll
      for (int g = 0; g < 4; ++g) {
        const float a = fmaxf(fmaxf(__int_as_float(acc[kt][4 * g]), __int_as_float(acc[kt][4 * g + 1])),
                              fmaxf(__int_as_float(acc[kt][4 * g + 2]), __int_as_float(acc[kt][4 * g + 3])));
        mx = fmaxf(mx, __fmul_rn(a, fabsf(fac.at(kt, g, 0))));
      }
    }
  } else {
    // a scale per key: the maximum of the products themselves (a masked score is -inf whatever its factor)
    mx = -INFINITY;
#pragma unroll
    for (int kt = 0; kt < 2; ++kt) {
#pragma unroll
      for (int v = 0; v < 16; v += 2)
        mx = fmaxf(fmaxf(mx, __fmul_rn(__int_as_float(acc[kt][v]), fabsf(fac.at(kt, v / 4, v % 4)))),
                   __fmul_rn(__int_as_float(acc[kt][v + 1]), fabsf(fac.at(kt, (v + 1) / 4, (v + 1) % 4))));
    }
  }
  {
    // the other half of the wavefront holds the other 32 keys of the same query
    const unsigned u = __float_as_uint(mx);
    const auto sw = __builtin_amdgcn_permlane32_swap(u, u, false, false);
    mx = fmaxf(__uint_as_float(sw[0]), __uint_as_float(sw[1]));
  }
  const float m_new = fmaxf(st.m_run, mx);
  // The static scale of P~ (Sec. 3.3: *448; *57344 or *127 for the other data types) is folded into the exponent:
  // E = scale * P~ = 2^(S - e), e = m - log2(scale).  Rounded to nearest, e could come out below m - log2(scale) and
  // the row's largest E above the scale - for scores beyond 2^19 far enough to overflow the 8-bit format, whose
  // conversion then gives NaN.  So m is first nudged upward by |m| 2^-22 (two to four units of its last place):
  // E <= scale whatever the roundings; the factor 2^-(2^-22 |m|) on P~ cancels in O / l.  The previous sums are
  // rescaled by the power of two of the offsets' difference (2^-inf = 0 on the first block), so O and l stay
  // sums under the current offset exactly.
  const float e_new = __fmaf_rn(fabsf(m_new), 0x1p-22f, m_new) -
                      (PVF == PV_INT8 ? LOG2_127 : (PVF == PV_E5M2 ? LOG2_57344 : LOG2_448));
  const float alpha = __builtin_amdgcn_exp2f(m_sub - e_new);      // m_sub: the offset of the previous block
  m_sub = e_new;
  st.m_run = m_new;
  return alpha;
}

// exp_group: 448 * P~ = 2^(S - m_sub) for the group (INT8 mode: S = sc * c, fused), its row-sum share
// added to ls, its FP8 codes written into word 4*KT + G of the P~ operand.
template <bool INT4, bool MASKED, int GM, int PVF, int KT, int G>
__device__ __forceinline__ void exp_group(const v16i (&acc)[2], const Factors<GM>& fac, float m_sub, v8i& pb,
                                          float& ls) {
  float e[4];
#pragma unroll
  for (int r = 0; r < 4; ++r) {
    const float x = __int_as_float(acc[KT][4 * G + r]);
    float arg;
    if constexpr (!fused_factor<INT4, GM>()) {
      arg = x - m_sub;
    } else {
      arg = __fmaf_rn(x, fac.at(KT, G, r), -m_sub);
      if constexpr (MASKED) arg = x == -INFINITY ? -INFINITY : arg;   // also when c = 0
    }
    e[r] = __builtin_amdgcn_exp2f(arg);
    ls += e[r];
  }
  int wd = __float_as_int(e[0]);   // any value: both halves are overwritten below
  if constexpr (PVF == PV_INT8) {
    // rint(127 P~) clipped to [0, 127] as bytes (the conversion is exact on the rounded values).  The clip
    // matters: for scores beyond 2^16 the rounding of m - log2(127) lets the row's largest term come out as
    // 127 * 2^(half an ulp of m) > 127.5, and a byte of 128 would be read as -128 by the integer MFMA.
#pragma unroll
    for (int r = 0; r < 4; ++r)
      wd = (int)__builtin_amdgcn_cvt_pk_u8_f32(rintf(fminf(e[r], INT8_PV_MAX)), (unsigned)r, (unsigned)wd);
  } else if constexpr (PVF == PV_E5M2) {
    wd = __builtin_amdgcn_cvt_pk_bf8_f32(e[0], e[1], wd, false);
    wd = __builtin_amdgcn_cvt_pk_bf8_f32(e[2], e[3], wd, true);
  } else {
    wd = __builtin_amdgcn_cvt_pk_fp8_f32(e[0], e[1], wd, false);
    wd = __builtin_amdgcn_cvt_pk_fp8_f32(e[2], e[3], wd, true);
  }
  pb[KT * 4 + G] = wd;
}

// Second half: the two-level accumulation of Sec. 3.4 on gfx950.  One v_mfma_f32_32x32x64_f8f6f4 has
// K = 64 = b_kv: the instruction sums the block's 64 FP8 products in its internal accumulator
// (level 1, confined to this block) and then adds its C operand in full FP32 (level 2: the
// cross-block accumulator O; measured - C passes through bit-exactly and C + product keeps FP32
// precision).  So O is the C/D operand, pre-scaled by alpha = 2^(m_old - m_new) only when some
// query of the wavefront actually moved its running max in this block.
template <int D>
__device__ __forceinline__ void block_rescale(RowState<D>& st, float alpha) {
  if (__builtin_amdgcn_ballot_w64(alpha != 1.0f) != 0) {
#pragma unroll
    for (int ct = 0; ct < D / 32; ++ct) {
#pragma unroll
      for (int v = 0; v < 16; ++v) st.O[ct][v] = __fmul_rn(alpha, st.O[ct][v]);
    }
  }
}
// With INT8 codes the block's product is an integer matrix product (two K = 32 instructions) into a
// fresh int32 accumulator - level 1 of Sec. 3.4 as the paper describes it - which is then converted and
// added to O in FP32 (level 2): 32 more vector instructions per channel tile and block.
template <int D, int CT, int PVF>
__device__ __forceinline__ void pv_step(RowState<D>& st, const v4i (&va)[2 * (D / 32)], const v8i& pb) {
  if constexpr (PVF == PV_INT8) {
    const v4i p0 = {pb[0], pb[1], pb[2], pb[3]}, p1 = {pb[4], pb[5], pb[6], pb[7]};
    v16i r;
#pragma unroll
    for (int v = 0; v < 16; ++v) r[v] = 0;
    r = __builtin_amdgcn_mfma_i32_32x32x32_i8(va[CT * 2 + 0], p0, r, 0, 0, 0);
    r = __builtin_amdgcn_mfma_i32_32x32x32_i8(va[CT * 2 + 1], p1, r, 0, 0, 0);
#pragma unroll
    for (int v = 0; v < 16; ++v) st.O[CT][v] = __fadd_rn(st.O[CT][v], (float)r[v]);
    return;
  }
  v8i a;
  const v4i a0 = va[CT * 2 + 0];
  const v4i a1 = va[CT * 2 + 1];
  a[0] = a0[0]; a[1] = a0[1]; a[2] = a0[2]; a[3] = a0[3];
  a[4] = a1[0]; a[5] = a1[1]; a[6] = a1[2]; a[7] = a1[3];
  // operand formats: 0 = E4M3, 1 = E5M2, for both V^ (A) and P^ (B)
  constexpr int FMT = PVF == PV_E5M2 ? 1 : 0;
  st.O[CT] = __builtin_amdgcn_mfma_scale_f32_32x32x64_f8f6f4(a, pb, st.O[CT], FMT, FMT, 0, 0, 0, 0);
  // The product is a 16-pass instruction, and a vector read of its result needs 20 wait states behind it.  The compiler fills
  // them in, but looks for the instruction only 19 back: a read that comes exactly 19 behind by itself gets nothing, and
  // returned old values of the registers written last (seen at a copy of O at the end of a loop body).  It counts an
  // asm statement as nothing, so this one makes every distance it leaves one longer than it thinks.  No measurable cost.
#if defined(__HIP_DEVICE_COMPILE__)
  asm volatile("s_nop 0" : "+v"(st.O[CT]));
#endif
}

// Wavefronts per SIMD the attention kernel is built for, by variant.  d = 128 with the default key groups: 3 (168
// registers: one block's scores live at a time, no software pipeline inside a wavefront - the other two wavefronts
// of the SIMD fill its waits; measured 8 - 9 % faster than 2 wavefronts with the score product of the next block
// pipelined into the exponentials of the current one).  The variants that hold more per-block state (a key scale
// per quad or per key, the INT8 P~V product) would spill at 168 registers and keep the pipelined form at 2.
// d = 64: half the accumulator, one more wavefront.  d = 256: 2 (the accumulator alone is 128 registers; 254 in all,
// two LDS stages of 29 KB so that two workgroups fit a CU; 2140 TOPS on the causal 8k case against 1254 for the
// pipelined form at one wavefront per SIMD, whose accumulators had to live in the second half of the register file).
#ifndef SAGE_OCC_D128
#define SAGE_OCC_D128 3
#endif
#ifndef SAGE_OCC_D64
#define SAGE_OCC_D64 4
#endif
#ifndef SAGE_OCC_D256
#define SAGE_OCC_D256 2
#endif
template <int D, int GM, int PVF> constexpr int attn_occupancy() {
  if (D == 256) return SAGE_OCC_D256;
  if (D == 128) return (GM == 0 && PVF != PV_INT8) ? SAGE_OCC_D128 : 2;
  return GM == 0 && PVF != PV_INT8 ? SAGE_OCC_D64 : (SAGE_OCC_D64 >= 3 ? 3 : 2);
}

// Global -> LDS copies without a register stop (the LDS-DMA form of the global load: lane l's
// 16 or 4 bytes land at LDS byte m0 + 16*l or m0 + 4*l).  Issued from inline assembly so that
// the wait for them is placed by hand - one vmcnt wait right before the barrier that publishes a
// stage - instead of in front of every later LDS read.  gbase is wavefront-uniform.
__device__ __forceinline__ void dma_b128(const void* gbase, unsigned voff, unsigned lds_byte) {
  unsigned m0_after;    // M0 is declared as a result, so the compiler knows the statement overwrites it
  asm volatile("s_mov_b32 m0, %1\n\ts_nop 0\n\tglobal_load_lds_dwordx4 %2, %3"
               : "={m0}"(m0_after) : "s"(lds_byte), "v"(voff), "s"(gbase) : "memory");
}
__device__ __forceinline__ void dma_b32(const void* gbase, unsigned voff, unsigned lds_byte) {
  unsigned m0_after;
  asm volatile("s_mov_b32 m0, %1\n\ts_nop 0\n\tglobal_load_lds_dword %2, %3"
               : "={m0}"(m0_after) : "s"(lds_byte), "v"(voff), "s"(gbase) : "memory");
}

// The 16-byte form for the lanes of `mask` alone (wavefront-uniform; none is allowed: then nothing is copied).
__device__ __forceinline__ void dma_b128_lanes(const void* gbase, unsigned voff, unsigned lds_byte, unsigned long long mask) {
  unsigned m0_after;
  unsigned long long all;
  asm volatile("s_mov_b32 m0, %2\n\ts_mov_b64 %1, exec\n\ts_mov_b64 exec, %5\n\ts_nop 0\n\t"
               "global_load_lds_dwordx4 %3, %4\n\ts_mov_b64 exec, %1"
               : "={m0}"(m0_after), "=&s"(all) : "s"(lds_byte), "v"(voff), "s"(gbase), "s"(mask) : "memory");
}
// A pointer that is the same in every lane, in scalar registers.
__device__ __forceinline__ const char* uniform_ptr(const char* p) {
  const unsigned long long u = (unsigned long long)p;
  const unsigned lo = __builtin_amdgcn_readfirstlane((unsigned)u), hi = __builtin_amdgcn_readfirstlane((unsigned)(u >> 32));
  return reinterpret_cast<const char*>((unsigned long long)hi << 32 | lo);
}

// An empty use of a register: the compiler must have the value complete (its load waited for) here.
__device__ __forceinline__ void use_now(int x) { asm volatile("" :: "v"(x)); }
__device__ __forceinline__ void use_now(float x) { asm volatile("" :: "v"(x)); }

// where query r of (batch b, head h) goes in the log-sum-exp output: [B, H, N], or [H, total_q] for a
// variable-length batch
__device__ __forceinline__ size_t lse_index(const AttnParams& p, const Seq& sq, int b, int h, int r) {
  if (p.seq.cu_q) return (size_t)h * (size_t)p.seq.cu_q[p.B] + sq.q0 + r;
  return ((size_t)b * p.H + h) * p.N + r;
}

}  // namespace sage
