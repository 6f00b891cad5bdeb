// Preprocessing kernels of the quantized attention forward pass (paper Sec. 3.1-3.3 and the
// "Preprocessing" line plus the first line of the outer loop of Algorithm 1): token means,
// smoothing, Delta-S, group quantization of Q and K, per-channel FP8 quantization of V.
// The passes stream Q, K and V once or twice each; after the loads it is the vector ALU work per
// element (and, for Delta-S, the FP64 matrix pipe) that sets their speed, so the quantizers avoid
// per-element divisions and per-element code packing.  Codes are written in the MFMA fragment
// order described in sage_common.h so that the attention kernel can move them with plain 16-byte
// copies.
#include "sage_quant.h"
#include "sage_attn.h"
#include <type_traits>

namespace sage {

// ------------------------------------------------------------------------------------------
// Column statistics: exact token sums of K (float64 accumulation of 16-bit values) and
// per-channel max |V| (Algorithm 1, "Preprocessing": mean(K) and the scale of psi_V).  Every
// workgroup writes the partial result of its STAT_ROWS tokens; the finalize kernels reduce the
// partials of a head (no atomics, nothing to clear beforehand).
constexpr int STAT_UNROLL = 4; // rows per thread in flight

// With the smooth-V option the first pass takes the exact token sums of V instead of max|V| (the
// maximum must be taken of the centred values, which needs the mean first: k_v_absmax below).
// (The bodies of the preprocessing kernels take their LDS from the kernel: one that runs two of them side by side overlays it.)
template <int D, bool SMOOTH_V> struct StatsLds {
  static constexpr int NRG = 256 / (D / 8);
  double sum[NRG][D], vsum[SMOOTH_V ? NRG : 1][D];
  float max[SMOOTH_V ? 1 : NRG][D];
};
template <bool BF16, int D, bool SMOOTH_V>
__device__ __forceinline__ void col_stats_block(StatsLds<D, SMOOTH_V>& lds, const BlockPos bp, const unsigned short* __restrict__ K,
                                                const unsigned short* __restrict__ V, double* __restrict__ k_sum,
                                                double* __restrict__ v_sum, unsigned* __restrict__ v_max, int Nq, int N,
                                                const TensorMap& km, const SeqMap& sm) {
  constexpr int NCG = D / 8, NRG = 256 / NCG;
  auto& s_sum = lds.sum; auto& s_vsum = lds.vsum; auto& s_max = lds.max;
  const int t = threadIdx.x, cg = t % NCG, rg = t / NCG;
  const HeadPos hp = head_pos(km, bp.y);
  const Seq sq = seq_of(sm, hp.b, Nq, N);
  const int r0 = bp.x * STAT_ROWS;
  const int r1 = min(r0 + STAT_ROWS, sq.nk);
  const size_t hbase = hp.base + sq.k0 * (size_t)km.sn;
  double acc[8], vacc[8];
  float mx[8];
#pragma unroll
  for (int e = 0; e < 8; ++e) { acc[e] = 0.0; vacc[e] = 0.0; mx[e] = 0.0f; }
  // STAT_UNROLL rows of K and of V are requested before the first is consumed: the pass is pure
  // streaming, and the bytes in flight per CU are what sets its bandwidth (rows past the end read
  // as zeros, which change neither a sum nor a maximum of magnitudes)
  for (int r = r0 + rg; r < r1; r += STAT_UNROLL * NRG) {
    uint4 rk[STAT_UNROLL], rv[STAT_UNROLL];
#pragma unroll
    for (int u = 0; u < STAT_UNROLL; ++u) {
      const int rr = r + u * NRG;
      rk[u] = rv[u] = make_uint4(0u, 0u, 0u, 0u);
      if (rr < r1) {
        const size_t row = row_offset(km, hbase, rr) + cg * 8;
        rk[u] = nt_load16(K + row);
        rv[u] = nt_load16(V + row);
      }
    }
#pragma unroll
    for (int u = 0; u < STAT_UNROLL; ++u) {
      float xk[8], xv[8];
      unpack8<BF16>(rk[u], xk);
      unpack8<BF16>(rv[u], xv);
#pragma unroll
      for (int e = 0; e < 8; ++e) {
        acc[e] += (double)xk[e];
        if constexpr (SMOOTH_V) vacc[e] += (double)xv[e]; else mx[e] = fmaxf(mx[e], fabsf(xv[e]));
      }
    }
  }
#pragma unroll
  for (int e = 0; e < 8; ++e) {
    s_sum[rg][cg * 8 + e] = acc[e];
    if constexpr (SMOOTH_V) s_vsum[rg][cg * 8 + e] = vacc[e]; else s_max[rg][cg * 8 + e] = mx[e];
  }
  __syncthreads();
  if (t < D) {
    double s = 0.0, sv = 0.0;
    float m = 0.0f;
    for (int g = 0; g < NRG; ++g) {
      s += s_sum[g][t];
      if constexpr (SMOOTH_V) sv += s_vsum[g][t]; else m = fmaxf(m, s_max[g][t]);
    }
    const size_t slot = ((size_t)bp.y * bp.nx + bp.x) * D + t;
    k_sum[slot] = s;
    if constexpr (SMOOTH_V) v_sum[slot] = sv;
    else v_max[slot] = __float_as_uint(m);
  }
}

template <bool BF16, int D, bool SMOOTH_V>
__global__ void __launch_bounds__(256) k_col_stats(const unsigned short* __restrict__ K,
                                                   const unsigned short* __restrict__ V,
                                                   double* __restrict__ k_sum, double* __restrict__ v_sum,
                                                   unsigned* __restrict__ v_max, int Nq, int N, TensorMap km,
                                                   SeqMap sm) {
  __shared__ StatsLds<D, SMOOTH_V> lds;
  col_stats_block<BF16, D, SMOOTH_V>(lds, block_pos(km), K, V, k_sum, v_sum, v_max, Nq, N, km, sm);
}

// Smooth-V option, second pass over V: per-channel max |fl32(V - mean(V))|.
template <bool BF16, int D>
__global__ void __launch_bounds__(256) k_v_absmax(const unsigned short* __restrict__ V,
                                                  const float* __restrict__ v_mean,
                                                  unsigned* __restrict__ v_max, int Nq, int N, TensorMap km,
                                                  SeqMap sm) {
  constexpr int NCG = D / 8, NRG = 256 / NCG;
  __shared__ float s_max[NRG][D];
  const int t = threadIdx.x, cg = t % NCG, rg = t / NCG;
  const BlockPos bp = block_pos(km);
  const HeadPos hp = head_pos(km, bp.y);
  const Seq sq = seq_of(sm, hp.b, Nq, N);
  const int r0 = bp.x * STAT_ROWS;
  const int r1 = min(r0 + STAT_ROWS, sq.nk);
  const size_t hbase = hp.base + sq.k0 * (size_t)km.sn;
  float mean[8], mx[8];
#pragma unroll
  for (int e = 0; e < 8; ++e) { mean[e] = v_mean[(size_t)bp.y * D + cg * 8 + e]; mx[e] = 0.0f; }
  for (int r = r0 + rg; r < r1; r += NRG) {
    float xv[8];
    load8<BF16>(V + row_offset(km, hbase, r) + cg * 8, xv);
#pragma unroll
    for (int e = 0; e < 8; ++e) mx[e] = fmaxf(mx[e], fabsf(__fsub_rn(xv[e], mean[e])));
  }
#pragma unroll
  for (int e = 0; e < 8; ++e) s_max[rg][cg * 8 + e] = mx[e];
  __syncthreads();
  if (t < D) {
    float m = 0.0f;
    for (int g = 0; g < NRG; ++g) m = fmaxf(m, s_max[g][t]);
    v_max[((size_t)bp.y * bp.nx + bp.x) * D + t] = __float_as_uint(m);
  }
}

// Partial results requested together where a workgroup reduces its head's (one round trip per batch instead of per chunk: whole calls of 128
// heads of 1024 tokens 94.7 -> 92.2 us, 16 of 3000 of 64 channels 66.2 -> 62.7, 8 of 5000 108.5 -> 102.8; batches of 8 and 16 the same, but
// 192 heads of 500 43.5 -> 42.4 with 4, 42.8 with 8, 43.5 with 16).
constexpr int SUM_BATCH = 4;
// the sum over a head's chunks of one channel (exact, whatever the order)
__device__ __forceinline__ double sum_partials(const double* __restrict__ part, size_t head, int nchunk, int d, int c) {
  const double* p = part + head * nchunk * d + c;
  double s = 0.0;
  for (int ch = 0; ch < nchunk; ch += SUM_BATCH) {
    double x[SUM_BATCH];
#pragma unroll
    for (int i = 0; i < SUM_BATCH; ++i) x[i] = p[(size_t)min(ch + i, nchunk - 1) * d];
#pragma unroll
    for (int i = 0; i < SUM_BATCH; ++i) s += ch + i < nchunk ? x[i] : 0.0;
  }
  return s;
}

// The LDS of two bodies of which a workgroup runs one.
template <class A, class B> union Overlay { A a; B b; __device__ Overlay() {} };

// k_mean = fl32(sum / N) (Eq. 2), delta_V = fl32(max|V| / 448) (Sec. 3.3); with the smooth-V option
// this call produces v_mean = fl32(sum / N) instead of delta_V, which k_finalize_vscale adds later.
// FIN_ENT (head, channel) entries per workgroup, FIN_PARTS threads each (256): thread part p sums chunks p, p + FIN_PARTS,
// ... (the sums are exact in float64, so their order does not matter) and the parts meet in LDS.  Many threads per
// entry because a long key range leaves many chunks (128 at 32 k keys) and a thread's loads are one round trip each.
constexpr int FIN_ENT = 16, FIN_PARTS = 16;
struct Finalize {
  const double *k_sum, *v_sum;
  const unsigned* v_max;
  float *k_mean, *v_mean, *v_scale;
  int n, Nq, N, d, Hkv, nchunk;
  SeqMap sm;
  float code_max;
  int smooth_k;
};
struct FinalizeLds {
  double k[FIN_PARTS][FIN_ENT], v[FIN_PARTS][FIN_ENT];
  float m[FIN_PARTS][FIN_ENT];
};
__device__ __forceinline__ void finalize_stats_block(FinalizeLds& lds, unsigned block, const Finalize& a) {
  const int e = threadIdx.x % FIN_ENT, part = threadIdx.x / FIN_ENT;
  const int i = block * FIN_ENT + e;
  double ks = 0.0, vs = 0.0;
  float vm = 0.0f;
  if (i < a.n) {
    const int head = i / a.d, c = i - head * a.d;
    const size_t p0 = (size_t)head * a.nchunk * a.d + c;
#pragma unroll 4
    for (int ch = part; ch < a.nchunk; ch += FIN_PARTS) {
      ks += a.k_sum[p0 + (size_t)ch * a.d];
      if (a.v_sum) vs += a.v_sum[p0 + (size_t)ch * a.d];
      else vm = fmaxf(vm, __uint_as_float(a.v_max[p0 + (size_t)ch * a.d]));
    }
  }
  lds.k[part][e] = ks; lds.v[part][e] = vs; lds.m[part][e] = vm;
  __syncthreads();
  if (part == 0 && i < a.n) {
    const int head = i / a.d;
    const int nk = seq_of(a.sm, (unsigned)(head / a.Hkv), a.Nq, a.N).nk;      // this sequence's key count
    ks = 0.0; vs = 0.0; vm = 0.0f;
#pragma unroll
    for (int q = 0; q < FIN_PARTS; ++q) {
      ks += lds.k[q][e];
      vs += lds.v[q][e];
      vm = fmaxf(vm, lds.m[q][e]);
    }
    a.k_mean[i] = nk > 0 && a.smooth_k ? (float)(ks / (double)nk) : 0.0f;   // smoothing of K off: mean 0
    if (a.v_sum) a.v_mean[i] = nk > 0 ? (float)(vs / (double)nk) : 0.0f;
    else a.v_scale[i] = __fdiv_rn(vm, a.code_max);
  }
}
__global__ void __launch_bounds__(256) k_finalize_stats(const Finalize a) {
  __shared__ FinalizeLds lds;
  finalize_stats_block(lds, blockIdx.x, a);
}
// Running statistics of a growing K / V (a KV cache that is appended to): the exact column sums of K and the column
// maxima of |V| are kept as state, a new chunk's partial results are added to them, and mean(K), delta_V of the whole
// are written.  Float64 sums of 16-bit values are exact, so the state after any sequence of chunks equals the one
// pass over everything, bit for bit.  fresh != 0: the state is initialised from this chunk.
// Workgroups of FIN_ENT entries with FIN_PARTS threads each, as in k_finalize_stats: a thread per entry took one round trip
// per eight chunks (k_finalize_vscale, 70 chunks of 96 heads of 64 channels: 21 us, now 5).
__global__ void __launch_bounds__(256) k_accumulate_stats(const double* __restrict__ k_sum, const unsigned* __restrict__ v_max,
                                   double* __restrict__ state_sum, float* __restrict__ state_max,
                                   float* __restrict__ k_mean, float* __restrict__ v_scale, int n, int d, int nchunk,
                                   int fresh, long long n_total, float code_max) {
  __shared__ double s_k[FIN_PARTS][FIN_ENT];
  __shared__ float s_m[FIN_PARTS][FIN_ENT];
  const int e = threadIdx.x % FIN_ENT, part = threadIdx.x / FIN_ENT;
  const int i = blockIdx.x * FIN_ENT + e;
  double ks = 0.0;
  float vm = 0.0f;
  if (i < n) {
    const int head = i / d, c = i - head * d;
    const size_t p0 = (size_t)head * nchunk * d + c;
#pragma unroll 4
    for (int ch = part; ch < nchunk; ch += FIN_PARTS) {
      ks += k_sum[p0 + (size_t)ch * d];
      vm = fmaxf(vm, __uint_as_float(v_max[p0 + (size_t)ch * d]));
    }
  }
  s_k[part][e] = ks; s_m[part][e] = vm;
  __syncthreads();
  if (part == 0 && i < n) {
    ks = fresh ? 0.0 : state_sum[i];
    vm = fresh ? 0.0f : state_max[i];
#pragma unroll
    for (int q = 0; q < FIN_PARTS; ++q) {
      ks += s_k[q][e];
      vm = fmaxf(vm, s_m[q][e]);
    }
    state_sum[i] = ks;
    state_max[i] = vm;
    k_mean[i] = n_total > 0 ? (float)(ks / (double)n_total) : 0.0f;
    v_scale[i] = __fdiv_rn(vm, code_max);
  }
}

__global__ void __launch_bounds__(256) k_finalize_vscale(const unsigned* __restrict__ v_max, float* __restrict__ v_scale, int n,
                                                         int d, int nchunk, float code_max) {
  __shared__ float s_m[FIN_PARTS][FIN_ENT];
  const int e = threadIdx.x % FIN_ENT, part = threadIdx.x / FIN_ENT;
  const int i = blockIdx.x * FIN_ENT + e;
  float vm = 0.0f;
  if (i < n) {
    const int head = i / d, c = i - head * d;
    const size_t p0 = (size_t)head * nchunk * d + c;
#pragma unroll 4
    for (int ch = part; ch < nchunk; ch += FIN_PARTS) vm = fmaxf(vm, __uint_as_float(v_max[p0 + (size_t)ch * d]));
  }
  s_m[part][e] = vm;
  __syncthreads();
  if (part == 0 && i < n) {
#pragma unroll
    for (int q = 0; q < FIN_PARTS; ++q) vm = fmaxf(vm, s_m[q][e]);
    v_scale[i] = __fdiv_rn(vm, code_max);
  }
}

// ------------------------------------------------------------------------------------------
// Fixed-point digits for the Delta-S product (the scheme is described at k_quant_k).
constexpr int DS_ND = 6;                         // digits per number
constexpr int DS_MAXPAIR = 6;                    // digit pairs (a, b) with a + b up to this are multiplied: 26 of 36

// A row's fixed point: up = 2^E with E = exponent(mx) + 3 of the row's largest magnitude mx, so that |x| < 2^(E-2), and the
// FP64 number whose addition leaves N = rint(x 2^(48-E)), plus 128 in each of its six bytes, in the low 48 mantissa bits.
// A row of zeros, or magnitudes of 2^125 and beyond (whose products overflow FP32 anyway), get up = 0: Delta-S = 0.
struct DsScale { double magic; float up; };
__device__ __forceinline__ DsScale ds_row_scale(float mx) {
  const unsigned eb = __float_as_uint(mx) >> 23;              // biased exponent (mx >= 0)
  const bool ok = mx > 0.0f && eb <= 251u;
  DsScale s;
  s.magic = __longlong_as_double((long long)(((unsigned long long)(((eb + 903u) << 20) | 0x88080u) << 32) | 0x80808080u));
  s.up = ok ? __uint_as_float((eb + 3u) << 23) : 0.0f;
  return s;
}
// The DS_ND digits of four numbers of a row, digit a of the four in the bytes of out[a]: x = 2^E sum_a n_a 2^(-8(a+1)) up to
// 2^(E-49), n_a in -128..127 (n_0 in -64..64).  The 128 added to every byte turns the bytes of a two's-complement number
// into signed digits - a byte of 128 and more carries into the next one - and comes off again by flipping its top bit.
// Two instructions cut a number, one addition and the widening in front of it, and 18 lay four numbers out; bit-field
// extracts of two rounded halves (six digits of 7 bits) took 16 per number.
__device__ __forceinline__ void ds_digits4(const float (&x)[4], double magic, unsigned (&out)[DS_ND]) {
  static_assert(DS_ND == 6, "48 bits");
  unsigned lo[4], hi[4];
#pragma unroll
  for (int j = 0; j < 4; ++j) {
    const unsigned long long b = (unsigned long long)__double_as_longlong((double)x[j] + magic);
    lo[j] = (unsigned)b; hi[j] = (unsigned)(b >> 32);
  }
  auto bytes01 = [](unsigned x1, unsigned x0) { return __builtin_amdgcn_perm(x1, x0, 0x05010400u); };   // byte 0 of both, byte 1 of both
  auto bytes23 = [](unsigned x1, unsigned x0) { return __builtin_amdgcn_perm(x1, x0, 0x07030602u); };
  auto low = [](unsigned x1, unsigned x0) { return __builtin_amdgcn_perm(x1, x0, 0x05040100u); };
  auto high = [](unsigned x1, unsigned x0) { return __builtin_amdgcn_perm(x1, x0, 0x07060302u); };
  const unsigned l01 = bytes01(lo[1], lo[0]), l23 = bytes01(lo[3], lo[2]), m01 = bytes23(lo[1], lo[0]), m23 = bytes23(lo[3], lo[2]),
                 h01 = bytes01(hi[1], hi[0]), h23 = bytes01(hi[3], hi[2]);
  out[5] = low(l23, l01) ^ 0x80808080u; out[4] = high(l23, l01) ^ 0x80808080u;
  out[3] = low(m23, m01) ^ 0x80808080u; out[2] = high(m23, m01) ^ 0x80808080u;
  out[1] = low(h23, h01) ^ 0x80808080u; out[0] = high(h23, h01) ^ 0x80808080u;
}

// Digits of one row of block means (DS_DIGITS), by one wavefront: `row` holds the D means (LDS or global), `digits`
// receives [digit a][channel] bytes, `scale` 2^E.
template <int D>
__device__ __forceinline__ void ds_slice_row(const float* row, unsigned char* __restrict__ digits, float* __restrict__ scale,
                                             int lane) {
  constexpr int PER = D / 64;                  // consecutive channels per lane
  float x[PER];
  float mx = 0.0f;
#pragma unroll
  for (int e = 0; e < PER; ++e) {
    x[e] = row[PER * lane + e];
    mx = fmaxf(mx, fabsf(x[e]));
  }
  mx = wave_max(mx);
  const DsScale sc = ds_row_scale(mx);
  if (lane == 0) *scale = sc.up;
  float y[4];
#pragma unroll
  for (int e = 0; e < 4; ++e) y[e] = x[e < PER ? e : 0];
  unsigned dg[DS_ND];
  ds_digits4(y, sc.magic, dg);
#pragma unroll
  for (int a = 0; a < DS_ND; ++a) {
    unsigned char* dst = digits + a * D + PER * lane;
    if constexpr (PER == 4) *reinterpret_cast<unsigned*>(dst) = dg[a];
    else if constexpr (PER == 2) *reinterpret_cast<unsigned short*>(dst) = (unsigned short)dg[a];
    else *dst = (unsigned char)dg[a];
  }
}

// ------------------------------------------------------------------------------------------
// KV head of query head bh (G query heads per KV head)
__device__ inline size_t kv_head(const TensorMap& qm, unsigned bh, int G) {
  const unsigned b = bh / (unsigned)qm.heads, h = bh - b * (unsigned)qm.heads;
  return (size_t)b * (qm.heads / G) + h / G;
}
// Arguments of the Q quantizers (the 8-bit one leaves the last five alone).
struct QuantQ {
  const unsigned short* q;
  float *q_mean, *q_scale;
  int8_t* q_codes;
  int N, Nk, nQb, block_groups, qg;
  TensorMap qm;
  SeqMap sm;
  float* q_corr;             // null, or where the row constants of the log-sum-exp go (needs mean(K))
  const float* k_mean;
  int G;
  float kappa;
  const float* head_scale;
  int stats_only, smooth_q;
  unsigned char* q_digits;
  float* q_dscale;
  const double* k_sum;       // not null: mean(K) is not there yet, these are the partial sums of its chunks
  int nchunk, smooth_k;
  int narrow;                // 8-bit, 64 channels: the NARROW map of quant_q8_block
};
// mean(K) of one channel, from k_mean or from the partial sums
template <int D>
__device__ __forceinline__ float q_kbar(const QuantQ& a, unsigned kv_head, int nk, int c) {
  if (!a.k_sum) return a.k_mean[(size_t)kv_head * D + c];
  return nk > 0 && a.smooth_k ? (float)(sum_partials(a.k_sum, kv_head, a.nchunk, D, c) / (double)nk) : 0.0f;
}
#define SAGE_QUANT_Q_ARGS                                                                                              \
  const unsigned short* __restrict__ Q = a.q; float* __restrict__ q_scale = a.q_scale;                                 \
  int8_t* __restrict__ q_codes = a.q_codes;                                                                            \
  const int N = a.N, Nk = a.Nk, nQb = a.nQb, block_groups = a.block_groups, qg = a.qg, G = a.G, stats_only = a.stats_only; \
  const TensorMap& qm = a.qm; const SeqMap& sm = a.sm; float* __restrict__ q_corr = a.q_corr;                          \
  const float* __restrict__ head_scale = a.head_scale; const float kappa = a.kappa

// The rows of a 128-query block as the Q quantizers hold them: wavefront w has rows 32 w .. 32 w + 31, in passes, and the lanes of a pass take
// the place of the lanes of the matrix operand that the codes are for, so that a wavefront's codes leave in runs of 128 and 256 bytes straight
// from its registers.  (As an image put together in LDS they cost a barrier, a pass through LDS and the LDS itself.)
struct QBlock { unsigned qb, bh; int n0, valid; size_t hbase; int nk; };
__device__ __forceinline__ QBlock q_block(const QuantQ& a, unsigned qb, unsigned bh) {
  QBlock b;
  b.qb = qb; b.bh = bh; b.n0 = (int)qb * BQ;
  const HeadPos hp = head_pos(a.qm, bh);
  const Seq sq = seq_of(a.sm, hp.b, a.N, a.Nk);
  b.valid = min(BQ, sq.n - b.n0);              // (none: a block past the end of a shorter sequence)
  b.hbase = hp.base + sq.q0 * (size_t)a.qm.sn;
  b.nk = sq.nk;
  return b;
}

// Q, 8-bit variant: pair-group quantization psi_Q(Q_i), no smoothing (the 8-bit kernel of the
// paper's "two kernel implementations" leaves Q as it is).  One workgroup per 128 queries of one
// (batch, head); a wavefront quantizes by itself.  Lane l of a pass holds row l % 16 and the 16-channel pieces l / 16 + 4 m, 32 bytes
// each: four lanes read 128 consecutive bytes, and a piece is 16 bytes of codes.  Both passes' rows are requested together.
// Against codes laid out in LDS, rows as 8 channels of 4 to 8 rows per thread and a byte extract per code: 32 heads of 8192 tokens 36 -> 24 us (100 MB:
// 4.2 TB/s).  Bound: the loads in flight - a workgroup loads, computes and stores in turn, and a chip's worth of them starts together
// (walking several blocks with the next one's rows requested ahead gained nothing: the 4-bit form 45 -> 51 us on 4096 blocks).
// NARROW, for 64-wide heads of long token-major rows, whose 128 bytes lie apart: 8 channels a lane and 8 rows a pass in four, so that every load takes whole
// runs (4 sequences of 64 heads of 2667 tokens 38.0 -> 31.7 us, of 17870 231 -> 215; the code image in LDS had 33.9 and 216).  Its four short chains cost
// small calls more than that is worth (two sequences of 64 heads of 300 tokens, 384 blocks, 5.3 -> 6.0, of 900, 1024 blocks, 8.2 -> 7.3).
template <int D, bool INT4> struct QuantQLds {               // (8-bit mode)
  alignas(16) float kbar[D];         // mean(K) of the KV head (log-sum-exp output only)
  float bmax[4];
};
template <bool BF16, int D, bool NARROW>
__device__ __forceinline__ void quant_q8_block(QuantQLds<D, false>& lds, const QBlock bl, const QuantQ& a) {
  SAGE_QUANT_Q_ARGS;
  constexpr int NM = NARROW ? 1 : D / 64, NL = NARROW ? 1 : 2;           // pieces of a row per lane, loads of a piece
  constexpr int NP = NARROW ? 4 : 2, RP = 32 / NP, PC = 8 * NL;          // passes, rows of a pass, channels of a piece
  constexpr int QMAX = 127;
  const int t = threadIdx.x, w = t >> 6, rr = NARROW ? (t >> 3) & 7 : t & 15, kc = NARROW ? t & 7 : (t >> 4) & 3;
  static_assert(!NARROW || D == 64, "eight lanes a row");
  const int qb = bl.qb, n0 = bl.n0, valid = bl.valid;
  const size_t bh = bl.bh, hbase = bl.hbase;
  if (valid <= 0) return;                     // a block past the end of a shorter sequence
  uint4 raw[NP][NM][NL];
#pragma unroll
  for (int p = 0; p < NP; ++p) {
    const int r = 32 * w + RP * p + rr;
    const unsigned short* src = Q + row_offset(qm, hbase, n0 + min(r, valid - 1)) + PC * kc;
#pragma unroll
    for (int m = 0; m < NM; ++m) {
#pragma unroll
      for (int i = 0; i < NL; ++i) raw[p][m][i] = nt_load16(src + 64 * m + 8 * i);
    }
  }
  if (q_corr) {
    if (t < D) lds.kbar[t] = q_kbar<D>(a, kv_head(qm, (unsigned)bh, G), bl.nk, t);
    __syncthreads();
  }
  // a row's largest magnitude: its pieces, then the lanes that share it
  auto row_max = [&](int p) {
    float mx = 0.0f;
#pragma unroll
    for (int m = 0; m < NM; ++m) {
#pragma unroll
      for (int i = 0; i < NL; ++i) {
        float x[8];
        unpack8<BF16>(raw[p][m][i], x);
#pragma unroll
        for (int e = 0; e < 8; ++e) mx = fmaxf(mx, fabsf(x[e]));
      }
    }
    if constexpr (NARROW) mx = group_max<8>(mx);
    else mx = butterfly_max<32>(butterfly_max<16>(mx));
    return 32 * w + RP * p + rr < valid ? mx : 0.0f;      // (the rows past the end are copies of the last one: their codes are 0)
  };
  float block_max = 0.0f;
  if (block_groups) {       // per-block granularity: one scale for the whole 128-query block
#pragma unroll
    for (int p = 0; p < NP; ++p) block_max = fmaxf(block_max, row_max(p));
    block_max = wave_max(block_max);
    if ((t & 63) == 0) lds.bmax[w] = block_max;
    __syncthreads();
    block_max = fmaxf(fmaxf(lds.bmax[0], lds.bmax[1]), fmaxf(lds.bmax[2], lds.bmax[3]));
  }
  int8_t* const slab = q_codes + (bh * nQb + qb) * q_slab_bytes(D, false);
#pragma unroll
  for (int p = 0; p < NP; ++p) {
    const int r = 32 * w + RP * p + rr;
    if (q_corr) {
      // kappa * <q_r, mean(K)>, the row constant that smoothing K drops from the scores (Sec. 3.1; needed only for the log-sum-exp
      // output): float64 products and sums, one rounding; runs of 8 channels, then neighbours in pairs
      double part[NM];
#pragma unroll
      for (int m = 0; m < NM; ++m) {
        double run[NL];
#pragma unroll
        for (int i = 0; i < NL; ++i) {
          float x[8];
          unpack8<BF16>(raw[p][m][i], x);
          run[i] = 0.0;
#pragma unroll
          for (int e = 0; e < 8; ++e) run[i] += (double)x[e] * (double)lds.kbar[PC * kc + 64 * m + 8 * i + e];
        }
        if constexpr (NARROW) part[m] = butterfly_sum<4>(butterfly_sum<2>(butterfly_sum<1>(run[0])));
        else part[m] = butterfly_sum<32>(butterfly_sum<16>(run[0] + run[1]));
      }
      double dot = part[0];
      if constexpr (NM == 2) dot = part[0] + part[1];
      if constexpr (NM == 4) dot = (part[0] + part[1]) + (part[2] + part[3]);
      if (kc == 0 && r < valid) q_corr[(bh * nQb + qb) * BQ + r] = (float)((double)kappa * dot);
    }
    float mx = row_max(p);                                   // per query; the pair shares the larger one unless qg == 1
    if (qg == 2) mx = butterfly_max<NARROW ? 8 : 1>(mx);
    if (block_groups) mx = block_max;
    const float delta = head_scale ? head_scale[bh] : __fdiv_rn(mx, (float)QMAX);
    if (kc == 0 && (qg == 1 || (r & 1) == 0)) q_scale[(bh * nQb + qb) * (BQ >> (qg - 1)) + (r >> (qg - 1))] = delta;   // qg is 1 or 2
    if (stats_only) continue;            // per-tensor scales, first pass: only the block maxima are wanted
    const CodeScale qs = code_scale(delta);
#pragma unroll
    for (int m = 0; m < NM; ++m) {
      float x[PC];
#pragma unroll
      for (int i = 0; i < NL; ++i) unpack8<BF16>(raw[p][m][i], x + 8 * i);
      if (valid < BQ) {
#pragma unroll
        for (int e = 0; e < PC; ++e) x[e] = r < valid ? x[e] : 0.0f;
      }
      unsigned c[PC];
      code_group_bytes<PC, QMAX>(x, delta, qs, c);
      int8_t* const to = slab + q_code_off(r, PC * kc + 64 * m, D);
      if constexpr (NARROW) *reinterpret_cast<uint2*>(to) = make_uint2(pack4(c), pack4(c + 4));
      else *reinterpret_cast<uint4*>(to) = pack16(c);
    }
  }
}

// Q, 4-bit variant: block mean, smoothing, pair-group quantization (Algorithm 1: q_bar_i =
// mean(Q_i), psi_Q(Q_i - q_bar_i)).  Two thread-to-data maps, joined through LDS:
//  - loading and the exact column sums of the block mean use a coalesced map (a thread owns 8 channels of BQ*D/2048
//    rows), and the raw 16-bit rows are parked in LDS;
//  - quantization uses the map the codes are consumed in, a pass at a time: a lane owns 32 consecutive channels of a row, one MFMA lane's
//    payload, or 64 (d = 256), so the maximum of a scale group is two lane exchanges away and the codes leave
//    through one FP32->FP6 conversion instead of per-element table look-ups and 6-bit shifts.  (32 channels a lane at d = 256 too, in four passes of 8 rows:
//    codes in runs of 64 and 128 bytes, 16 heads of 13526 tokens, four sequences, token-major, 159 us, with 64 146, from an image in LDS 159.)
// LDS rows are kept as 16-byte chunks in an order by the row's number, which spreads the chunk that a pass reads of every row over all
// banks.  LDS: the raw rows (32 KB at d = 128) and one row of column sums per wavefront (the row groups of a wavefront are summed by
// lane exchanges first) - 37 KB, so that four workgroups share a CU and their loads, arithmetic and stores overlap.
// With the passes and no code image in LDS: 2 heads of 256 tokens (with the statistics) 5.05 -> 4.45 us, 64
// heads of 512 9.4 -> 8.8, 16 of 8192 of 256 channels 29.2 -> 28.1, 128 of 4096 42 to 45 (185 MB: 4.1 to 4.4 TB/s): loads and parking alone 29, column
// sums 4, quantization 6, stores 4.  (Rows read a second time instead of parked, five workgroups per CU: 48.)
template <int D> struct QuantQLds<D, true> {
  uint4 raw[BQ * (D / 8)];           // the raw rows
  double sum[4][D];                  // column sums, one row per wavefront
  alignas(16) float mean[D];
  alignas(16) float kbar[D];         // mean(K) of the KV head (log-sum-exp output only)
  float bmax[4];
  int odd_mean;                      // some column sum of the block is not finite
};
template <bool BF16, int D>
__device__ __forceinline__ void quant_q4_block(QuantQLds<D, true>& lds, const QBlock bl, const QuantQ& a) {
  SAGE_QUANT_Q_ARGS;
  float *__restrict__ q_mean = a.q_mean, *__restrict__ q_dscale = a.q_dscale;
  unsigned char* __restrict__ q_digits = a.q_digits;
  const int smooth_q = a.smooth_q;
  constexpr int NCG = D / 8, NRG = 256 / NCG, RPT = BQ / NRG;   // load map: RPT rows x 8 channels
  constexpr int CPL = D == 256 ? 64 : 32;                        // quantization map: channels per lane, lanes per row, and RP rows of a
  constexpr int NPC = D / CPL, RP = 64 / NPC, NPASS = 32 / RP;   // wavefront's 32 in a pass
  constexpr int QMAX = 7;
  auto& s_raw = lds.raw; auto& s_sum = lds.sum; auto& s_mean = lds.mean; auto& s_kbar = lds.kbar; auto& s_bmax = lds.bmax;
  auto chunk_at = [](int r, int c) { return r * NCG + (c ^ (D == 64 ? (r >> 1) & 7 : r & 15)); };
  const int t = threadIdx.x, cg = t % NCG, rg = t / NCG;
  const int qb = bl.qb, n0 = bl.n0, valid = bl.valid;
  const size_t bh = bl.bh, hbase = bl.hbase;
  if (valid <= 0) return;                     // a block past the end of a shorter sequence
  if (t == 0) lds.odd_mean = 0;
  uint4 raw[RPT];
  {
#pragma unroll
    for (int i = 0; i < RPT; ++i) {
      const int r = rg * RPT + i;
      raw[i] = r < valid ? nt_load16(Q + row_offset(qm, hbase, n0 + r) + cg * 8)
                         : make_uint4(0u, 0u, 0u, 0u);                  // padded rows are zero
    }
    double cs[8];
#pragma unroll
    for (int e = 0; e < 8; ++e) cs[e] = 0.0;
    // (fetched now, under the loads of the rows: read from global memory where it is used, in front of every 8 channels of
    // every row, it was a round trip each)
    if (q_corr && t < D) s_kbar[t] = q_kbar<D>(a, kv_head(qm, (unsigned)bh, G), bl.nk, t);
#pragma unroll
    for (int i = 0; i < RPT; ++i) {
      const int r = rg * RPT + i;
      s_raw[chunk_at(r, cg)] = raw[i];
      float x8[8];
      unpack8<BF16>(raw[i], x8);
#pragma unroll
      for (int e = 0; e < 8; ++e) cs[e] += (double)x8[e];
    }
    // a wavefront holds 64 / NCG row groups (lane = (rg % (64 / NCG)) * NCG + cg): summed by lane exchanges first
    // (float64 sums of 16-bit values are exact: the order of the additions does not matter)
#pragma unroll
    for (int e = 0; e < 8; ++e) {
      if constexpr (NCG == 8) cs[e] = butterfly_sum<8>(cs[e]);
      if constexpr (NCG <= 16) cs[e] = butterfly_sum<16>(cs[e]);
      cs[e] = butterfly_sum<32>(cs[e]);
    }
    if ((t & 63) < NCG) {
#pragma unroll
      for (int e = 0; e < 8; ++e) s_sum[t >> 6][cg * 8 + e] = cs[e];
    }
  }
  __syncthreads();
  if (t < D) {
    double sm = 0.0;
    for (int g = 0; g < 4; ++g) sm += s_sum[g][t];
    if (!(fabs(sm) < (double)INFINITY)) lds.odd_mean = 1;
    const float m = smooth_q ? (float)(sm / (double)valid) : 0.0f;   // smoothing of Q off: mean 0
    s_mean[t] = m;
    q_mean[(bh * nQb + qb) * D + t] = m;
  }
  __syncthreads();
  const int lane = t & 63, w = t >> 6, rr = lane % RP, piece = lane / RP, c0 = CPL * piece;
  const bool odd = lds.odd_mean != 0;
  auto row_of = [&](int p) { return 32 * w + RP * p + rr; };
  // kappa * <q_r, mean(K)> per row (the log-sum-exp output only): float64, runs of D / 4 channels one after the other, then neighbours in
  // pairs.  A lane's channels are one run, or two (d = 64).
  constexpr int RUN = D / 4, RUNS = CPL / RUN;
  // the lane's channels of row r, centred (a row past the end stays zero)
  auto load_row = [&](int r, float (&x)[CPL], double (&run)[RUNS], bool dots) {
#pragma unroll
    for (int j = 0; j < CPL / 8; ++j) {
      unpack8<BF16>(s_raw[chunk_at(r, CPL / 8 * piece + j)], &x[8 * j]);
      if (dots) {
        const float4 b0 = *reinterpret_cast<const float4*>(&s_kbar[c0 + 8 * j]);
        const float4 b1 = *reinterpret_cast<const float4*>(&s_kbar[c0 + 8 * j + 4]);
        const float kb[8] = {b0.x, b0.y, b0.z, b0.w, b1.x, b1.y, b1.z, b1.w};
        double& dot = run[RUNS == 2 ? j / 2 : 0];
        if (8 * j % RUN == 0) dot = 0.0;
#pragma unroll
        for (int e = 0; e < 8; ++e) dot += (double)x[8 * j + e] * (double)kb[e];
      }
      const float4 m0 = *reinterpret_cast<const float4*>(&s_mean[c0 + 8 * j]);
      const float4 m1 = *reinterpret_cast<const float4*>(&s_mean[c0 + 8 * j + 4]);
      const float mean[8] = {m0.x, m0.y, m0.z, m0.w, m1.x, m1.y, m1.z, m1.w};
#pragma unroll
      for (int e = 0; e < 8; ++e) x[8 * j + e] = __fsub_rn(x[8 * j + e], mean[e]);
    }
    if (valid < BQ) {
#pragma unroll
      for (int e = 0; e < CPL; ++e) x[e] = r < valid ? x[e] : 0.0f;
    }
  };
  auto row_max = [&](const float (&x)[CPL]) {
    float mx = 0.0f;
#pragma unroll
    for (int e = 0; e < CPL; ++e) mx = fmaxf(mx, fabsf(x[e]));
    if constexpr (NPC == 4) mx = butterfly_max<16>(mx);
    return butterfly_max<32>(mx);
  };
  // per-block granularity, one scale for the whole 128-query block, and the first pass of per-tensor scales, which only want the largest of the head's:
  // from the values as they were loaded.  (Read out of LDS, and their maxima formed row by row: 4 sequences of 8 heads of 214 tokens of 256 channels,
  // with the statistics, 10.9 us, this way 9.2; two passes of per-tensor scales, 4 x 32 heads of 2591 of 128, 30.4 each and 25.4.)
  float block_max = 0.0f;
  if ((block_groups && !head_scale) || stats_only) {
    float mean[8];
#pragma unroll
    for (int e = 0; e < 8; ++e) mean[e] = s_mean[8 * cg + e];
#pragma unroll
    for (int i = 0; i < RPT; ++i) {
      float x8[8];
      unpack8<BF16>(raw[i], x8);
      float mx = 0.0f;
#pragma unroll
      for (int e = 0; e < 8; ++e) mx = fmaxf(mx, fabsf(__fsub_rn(x8[e], mean[e])));
      if (rg * RPT + i < valid) block_max = fmaxf(block_max, mx);
    }
    block_max = wave_max(block_max);
    if (lane == 0) s_bmax[w] = block_max;
    __syncthreads();
    block_max = fmaxf(fmaxf(s_bmax[0], s_bmax[1]), fmaxf(s_bmax[2], s_bmax[3]));
    if (stats_only) {                    // (no log-sum-exp in this pass: the other one writes the row constants)
      if (t < (BQ >> (qg - 1))) q_scale[(bh * nQb + qb) * (BQ >> (qg - 1)) + t] = __fdiv_rn(block_max, (float)QMAX);
      return;
    }
  }
  uint8_t* const slab = reinterpret_cast<uint8_t*>(q_codes + (bh * nQb + qb) * q_slab_bytes(D, true));
#pragma unroll
  for (int p = 0; p < NPASS; ++p) {
    const int r = row_of(p);
    float x[CPL];
    double run[RUNS];
    load_row(r, x, run, q_corr != nullptr);
    if (q_corr) {
      double dot = run[0];
      if constexpr (RUNS == 2) dot = run[0] + run[1];
      if constexpr (NPC == 4) dot = butterfly_sum<16>(dot);
      dot = butterfly_sum<32>(dot);
      if (piece == 0 && r < valid) q_corr[(bh * nQb + qb) * BQ + r] = (float)((double)kappa * dot);
    }
    float mx = block_max;
    if (!block_groups && !head_scale) {
      mx = row_max(x);                                         // per query; the pair shares the larger one unless qg == 1
      if (qg == 2) mx = butterfly_max<1>(mx);
    }
    const float delta = head_scale ? head_scale[bh] : __fdiv_rn(mx, (float)QMAX);
    if (piece == 0 && (qg == 1 || (r & 1) == 0))   // qg is 1 or 2
      q_scale[(bh * nQb + qb) * (BQ >> (qg - 1)) + (r >> (qg - 1))] = delta;
    CodeScale qs = code_scale(delta);
    qs.fast = qs.fast && !odd;           // (the exact form makes 0 of NaN)
#pragma unroll
    for (int pl = 0; pl < CPL / 32; ++pl) {                    // (one MFMA lane's payload, or the two lane halves of one operand)
      Codes32 cd;
      code_group<32, QMAX>(&x[32 * pl], delta, qs, [&](int e, float c) { cd.set(e, c); });
      const v6u pw = cd.pack();
      int lane_m, e0;
      uint8_t* const op = slab + q_op6(r, c0 + 32 * pl, D, &lane_m, &e0);
      *reinterpret_cast<uint4*>(op + 16 * lane_m) = make_uint4(pw[0], pw[1], pw[2], pw[3]);
      *reinterpret_cast<uint2*>(op + 1024 + 8 * lane_m) = make_uint2(pw[4], pw[5]);
    }
  }
  // the block mean cut into digits for the Delta-S product: by one wavefront, where nobody waits for it any more (done in
  // front of the quantization it held up the other three: 4096 blocks of d = 128 48 us, now 45)
  if (q_digits && t >= 192)
    ds_slice_row<D>(s_mean, q_digits + (bh * nQb + qb) * (size_t)(DS_ND * D), q_dscale + (bh * nQb + qb), t - 192);
}

template <bool BF16, bool INT4, int D>
__device__ __forceinline__ void quant_q_block(QuantQLds<D, INT4>& lds, const QBlock bl, const QuantQ& a) {
  if constexpr (INT4) quant_q4_block<BF16, D>(lds, bl, a);
  else if constexpr (D == 64) { if (a.narrow) quant_q8_block<BF16, D, true>(lds, bl, a); else quant_q8_block<BF16, D, false>(lds, bl, a); }
  else quant_q8_block<BF16, D, false>(lds, bl, a);
}
// The first fin_rows rows of the grid finish the statistics (finalize_stats_block) under the quantization of Q.
template <bool BF16, bool INT4, int D>
__global__ void __launch_bounds__(256, D == 256 ? 2 : 4) k_quant_q(const QuantQ a, const Finalize f, const unsigned fin_rows) {
  __shared__ Overlay<QuantQLds<D, INT4>, FinalizeLds> lds;
  if (blockIdx.y < fin_rows) {
    finalize_stats_block(lds.b, blockIdx.y * gridDim.x + blockIdx.x, f);
    return;
  }
  const unsigned y = blockIdx.y - fin_rows;
  quant_q_block<BF16, INT4, D>(lds.a, a.qm.heads_inner ? q_block(a, y, blockIdx.x) : q_block(a, blockIdx.x, y), a);
}

// ------------------------------------------------------------------------------------------
// K: smoothing by the token mean, group quantization (runs of 16 keys by default) and, in the int4
// mode, Delta-S.
// (Algorithm 1: psi_K(K_j) after K = K - mean(K); Sec. 3.1: Delta-S = q_bar_i . gamma(K)^T.)
//
// One workgroup per 64 keys of one (batch, KV head); wavefront w owns keys 16w..16w+15, which
// is exactly one default quantization group.  Lane l holds key 16w + l%16 and the D/4 consecutive
// channels (D/4)*(l/16) .. +D/4-1, i.e. the wavefront reads 16 whole rows as one contiguous
// piece.  That is also the B-operand shape of the 16x16x4 FP64 MFMA (lane l supplies
// B[k = l/16][column l%16]) once contraction slot (step cs, k = l/16) is assigned channel
// (D/4)*(l/16) + cs - any assignment is valid as long as the A operand uses the same one - so
// the smoothed keys feed the Delta-S product straight from the registers they were quantized in.
//
// Delta-S: D[i, t] = fl32(kappa * <q_bar_i, gamma(K)_t>), the inner product formed exactly (or in float64) so that
// the value does not depend on summation order: a small GEMM [nQb x d] . [d x 64] per query head of the KV group,
// walked 16 query blocks (a step) at a time, their rows in one half of an LDS buffer while the next step's arrive for the other;
// three forms, template parameter DSM below.  The FP64 form:
// v_mfma_f64_16x16x4_f64 sustains about 70 TFLOP/s on the whole chip and, unlike the low-precision matrix
// instructions, does not run concurrently with other vector work of the SIMD, so it costs its own matrix time
// (2*nQb*N*d flops per head) on top of the quantization.
typedef double v4d __attribute__((ext_vector_type(4)));

constexpr int DS_ROWS = 16;     // block means per step of the Delta-S product: one tile of the 16-row matrix instructions

// How the Delta-S product is formed (template parameter DSM of k_quant_k):
//   DS_DIGITS  both factors cut into signed bytes of a fixed-point number and multiplied byte by byte on the INT8
//              matrix instruction: exact integer sums, recombined in float64 (the default),
//   DS_FP32    v_mfma_f32_16x16x4_f32: faster still, approximate (an option of the boundary),
//   DS_FP64    v_mfma_f64_16x16x4_f64: the reference form (an option of the boundary).
//
// DS_DIGITS.  A row x of d numbers (a block mean q_bar_i, or a smoothed key) with largest magnitude below 2^(E-2) is
// written x_c = 2^E sum_a n_a[c] 2^(-8(a+1)) + rest, a = 0..5, with digits that fit a signed byte (ds_digits4); the rest is
// zero for every x_c whose exponent is within 21 of the row's largest (smaller ones lose what lies below 2^(E-48)).  Then
//   <x, y> = 2^(Ex+Ey) sum_{a,b} 2^(-8(a+b+2)) sum_c n_a[c] m_b[c],
// the inner sums are integers below 2^21 (d = 128) that v_mfma_i32_16x16x64_i8 forms exactly, pairs with the same a + b share
// an accumulator (below 2^24), and the pairs with a + b > 6 are left out: together less than 2^-49 of
// |x|_max |y|_max d.  The result agrees with the float64 inner product far below its FP32 rounding, at a quarter of
// the FP64 instruction's time, and - being INT8 matrix work - it runs alongside the vector work of the quantizers.
// Bound: for a few rows vector issue (four cycles an instruction, whatever its class, once the wavefronts of a SIMD are out of
// step), which the cutting of the keys and the joining of the accumulators set; for many the chain of a step, loads, matrix
// instructions, joining, one barrier: 32 heads of 32768 tokens, causal, vector issue 56 % and matrix pipe 58 % busy; 16 heads of 8192
// tokens of 256 channels, two wavefronts per SIMD, 46 % and 29 %.
enum { DS_DIGITS = 0, DS_FP32 = 1, DS_FP64 = 2 };

// Arguments of the K and V quantizers.  Where the statistics pass left partial results that nobody has reduced (k_sum, v_max
// not null: the launch that covers both, k_quant_kv), every workgroup reduces its head's and the first one writes
// mean(K) and delta_V for the attention kernel.
struct QuantKV {
  const unsigned short *k, *v;
  float *k_mean, *v_scale;
  const float* v_mean;
  float* k_scale;
  int8_t* k_codes;
  uint8_t* v_codes;
  const float* q_mean;
  float* delta_s;
  int Nq, Nk, nKb, nQb, G;
  float kappa;
  int block_groups, kg, causal;
  TensorMap km;
  SeqMap sm;
  const float* head_scale;
  int stats_only, zero_ds;
  const unsigned char* q_digits;
  const float* q_dscale;
  const double* k_sum;
  const unsigned* v_max;
  int nchunk, smooth_k;
  float code_max;
  int mixed;                 // K and V in one launch: both on every XCD
  int bounded;               // delta_V was taken from these values
  int parts;                 // workgroups per key block of K (z of the grid)
};

template <int D, bool INT4, int DSM, bool REDUCE> struct QuantKLds {
  static constexpr bool DSD = INT4 && DSM == DS_DIGITS;
  // LDS row of staged block means: channel c sits at column c + 16*(c / 32) when D = 128, so the
  // 32 lanes of a half-wavefront (16 rows x 2 channel groups) hit 32 different banks (odd stride)
  static constexpr int SQW = D + (D >= 128 ? 48 : 0) + 1;
  // DS_DIGITS: a staged row is its DS_ND digit planes of D bytes; 16 bytes of padding make the 16 rows of an operand read
  // start in 16 different bank groups
  static constexpr int ROWB = DS_ND * D + 16;
  uint4 codes[k_block_bytes(D, INT4) / 16];        // the block's packed image
  float q[INT4 && !DSD ? 2 * DS_ROWS : 1][SQW];
  alignas(16) unsigned char qd[DSD ? 2 * DS_ROWS : 1][DSD ? ROWB : 16];
  double qs[DSD ? 2 * DS_ROWS : 1];                // 2^E of the staged rows
  alignas(16) float kmean[REDUCE ? D : 4];
  float bmax[4];
};
template <bool BF16, bool INT4, int D, int DSM = DS_DIGITS, bool REDUCE = false>
__device__ __forceinline__ void quant_k_block(QuantKLds<D, INT4, DSM, REDUCE>& lds, const BlockPos bp, const QuantKV& a, const int z = 0) {
  const unsigned short* __restrict__ K = a.k;
  float* __restrict__ k_scale = a.k_scale; int8_t* __restrict__ k_codes = a.k_codes;
  const float* __restrict__ q_mean = a.q_mean; float* __restrict__ delta_s = a.delta_s;
  const int Nq = a.Nq, Nmax = a.Nk, nKb = a.nKb, nQb = a.nQb, G = a.G, block_groups = a.block_groups, kg = a.kg, causal = a.causal;
  const float kappa = a.kappa; const TensorMap& km = a.km; const SeqMap& sm = a.sm;
  const float* __restrict__ head_scale = a.head_scale; const int stats_only = a.stats_only, zero_ds = a.zero_ds;
  const unsigned char* __restrict__ q_digits = a.q_digits; const float* __restrict__ q_dscale = a.q_dscale;
  constexpr bool DS32 = DSM == DS_FP32, DSD = INT4 && DSM == DS_DIGITS;
  constexpr int CPL = D / 4;                       // channels per lane (32 or 16)
  constexpr int QMAX = INT4 ? 7 : 127;
  constexpr int PADSH = D == 256 ? 6 : 5;          // 16 columns of padding after every 32 (d = 128) / 64 (d = 256) channels
  auto& s_codes = lds.codes; auto& s_q = lds.q; auto& s_qd = lds.qd; auto& s_qs = lds.qs; auto& s_kmean = lds.kmean; auto& s_bmax = lds.bmax;
  const int t = threadIdx.x, lane = t & 63, w = t >> 6;
  const int r16 = lane & 15, k4 = lane >> 4;
  const int kb = bp.x;
  const size_t bhkv = bp.y;
  const int n0 = kb * BKV;
  const int r = 16 * w + r16, c0 = CPL * k4;
  // this sequence's key count N, query-block count nQs and causal offset (the slabs keep the
  // strides nQb, nKb of the longest sequence)
  const HeadPos hp = head_pos(km, bp.y);
  const Seq sq = seq_of(sm, hp.b, Nq, Nmax);
  const int N = sq.nk, coff = sq.coff;
  const int nQs = (sq.n + BQ - 1) / BQ;
  if (n0 >= N) return;                             // a block past the end of a shorter sequence

  // The rows of the Delta-S product - the block means of the G query heads that share this KV head, from the first query block
  // that sees a key of this block on (under a causal mask block i does if 128 i + 127 + coff >= its first key) - are numbered
  // through all the heads and taken 16 at a time.  Which step a row sits in changes nothing in its value.
  const int i0 = causal ? min(max(n0 - coff, 0) / BQ, nQs) : 0;
  const int nr = nQs - i0, nrow = INT4 ? G * nr : 0;
  const int bh0 = (int)bhkv * G;
  const float inv_nr = __builtin_amdgcn_rcpf((float)max(nr, 1));
  // Of the steps this workgroup takes part `part` of a.parts (k_parts); the first one has the codes and scales too.  (Digit form only: with the others in it
  // their loops are compiled differently, 64 on 4 heads of 8989 tokens of 256 channels, FP32 form, 290 -> 305 us.)
  const int part = DSD ? z : 0, steps = (nrow + DS_ROWS - 1) / DS_ROWS;
  const int row0 = DSD ? DS_ROWS * (int)((unsigned)part * (unsigned)steps / (unsigned)a.parts) : 0;
  const int row_end = DSD ? min(nrow, DS_ROWS * (int)((unsigned)(part + 1) * (unsigned)steps / (unsigned)a.parts)) : nrow;
  if (part > 0 && row0 >= row_end) return;
  // A step's rows: nr >= 16 leaves room for one change of head, `cut` rows of the current one and then the next one's;
  // shorter heads are told apart by a division per row.
  struct Step { int R, base, next, cut; };         // first row, its place in the [B H][nQb] arrays, that of the next head's first row, cut
  auto step_at = [&](int R, int g, int i) { return Step{R, (bh0 + g) * nQb + i, (bh0 + g + 1) * nQb + i0, nQs - i}; };
  const bool few = nr < DS_ROWS;
  auto step_row = [&](const Step& q, int rr) {     // place of row rr of the step, or -1 for an empty row
    if (q.R + rr >= nrow) return -1;
    if (few) {
      // (R + 1/2) / nr never comes within rounding distance of an integer for the less than 2^21 rows there can be here
      const int R = q.R + rr, g = (int)(((float)R + 0.5f) * inv_nr);
      return (bh0 + g) * nQb + i0 + (R - g * nr);
    }
    return rr < q.cut ? q.base + rr : q.next + (rr - q.cut);
  };
  constexpr int NCH = DS_ND * D / 16;              // 16-byte pieces of a row of digits
  constexpr int QPD = (DS_ROWS * NCH + 255) / 256;         // ... per thread per step
  constexpr int QPT = (DS_ROWS * (D / 4) + 255) / 256;     // float4 pieces of the means per thread per step (the other forms)
  float4 qpre[DSD ? 1 : QPT];
  uint4 dpre[DSD ? QPD : 1];
  float spre = 0.0f;
  // (a step within one head: consecutive rows of the arrays)
  auto plain_step = [&](const Step& q) { return !few && q.cut >= DS_ROWS && nrow - q.R >= DS_ROWS; };
  auto load_q = [&](const Step& q) {
    if constexpr (DSD) {
      if (plain_step(q)) {
        const uint4* src = reinterpret_cast<const uint4*>(q_digits + (size_t)(unsigned)q.base * (DS_ND * D));
#pragma unroll
        for (int k = 0; k < QPD; ++k) {
          if ((k + 1) * 256 <= DS_ROWS * NCH || t + k * 256 < DS_ROWS * NCH) dpre[k] = src[(unsigned)(t + k * 256)];
        }
        if (t < DS_ROWS) spre = q_dscale[(unsigned)(q.base + t)];
        return;
      }
      int tt = t;
      asm volatile("" : "+v"(tt));       // (what this path needs is formed here: kept through the loop, it cost registers)
#pragma unroll
      for (int k = 0; k < QPD; ++k) {
        const int idx = tt + k * 256, rr = idx / NCH, ch = idx % NCH;
        const int row = rr < DS_ROWS ? step_row(q, rr) : -1;
        dpre[k] = row >= 0 ? *reinterpret_cast<const uint4*>(q_digits + (size_t)row * (DS_ND * D) + 16 * ch)
                           : make_uint4(0u, 0u, 0u, 0u);
      }
      if (t < DS_ROWS) {
        const int row = step_row(q, t);
        spre = row >= 0 ? q_dscale[row] : 0.0f;
      }
    } else {
#pragma unroll
      for (int k = 0; k < QPT; ++k) {
        const int idx = t + k * 256, rr = idx / (D / 4), c4 = idx % (D / 4);
        const int row = rr < DS_ROWS ? step_row(q, rr) : -1;
        qpre[k] = row >= 0 ? *reinterpret_cast<const float4*>(q_mean + (size_t)row * D + 4 * c4)
                           : make_float4(0.f, 0.f, 0.f, 0.f);
      }
    }
  };
  auto store_q = [&](int half) {                   // into one of the two halves of the LDS buffer
    if constexpr (DSD) {
#pragma unroll
      for (int k = 0; k < QPD; ++k) {
        const int idx = t + k * 256, rr = idx / NCH, ch = idx % NCH;
        if (DS_ROWS * NCH % 256 == 0 || rr < DS_ROWS) *reinterpret_cast<uint4*>(&s_qd[half * DS_ROWS + rr][16 * ch]) = dpre[k];
      }
      if (t < DS_ROWS) s_qs[half * DS_ROWS + t] = (double)spre;
    } else {
#pragma unroll
      for (int k = 0; k < QPT; ++k) {
        const int idx = t + k * 256, rr = idx / (D / 4), c4 = idx % (D / 4);
        const int col = 4 * c4 + (D >= 128 ? 16 * ((4 * c4) >> PADSH) : 0);
        float* dst = &s_q[half * DS_ROWS + rr][col];
        dst[0] = qpre[k].x; dst[1] = qpre[k].y; dst[2] = qpre[k].z; dst[3] = qpre[k].w;
      }
    }
  };
  // the K rows are requested first, then the first step's block means, so that the round trips overlap
  const size_t hbase = hp.base + sq.k0 * (size_t)km.sn;
  const unsigned short* krow = K + row_offset(km, hbase, min(n0 + r, N - 1)) + c0;
  uint4 kraw[CPL / 8];
#pragma unroll
  for (int p = 0; p < CPL / 8; ++p) kraw[p] = *reinterpret_cast<const uint4*>(krow + 8 * p);
  int g = part > 0 ? row0 / max(nr, 1) : 0, i = i0 + row0 - g * nr;       // head and query block of the step's first row
  Step step = step_at(row0, g, i);
  if constexpr (INT4) load_q(step);

  // mean(K) of this head: reduced by the statistics pass, or here
  if constexpr (REDUCE) {
    if (t < D) {
      const float m = a.smooth_k ? (float)(sum_partials(a.k_sum, (size_t)bhkv, a.nchunk, D, t) / (double)N) : 0.0f;
      s_kmean[t] = m;
      if (kb == 0 && part == 0) a.k_mean[bhkv * D + t] = m;
    }
    __syncthreads();
  }
  auto mean4 = [&](int c) {
    return REDUCE ? *reinterpret_cast<const float4*>(&s_kmean[c]) : *reinterpret_cast<const float4*>(a.k_mean + bhkv * D + c);
  };

  float x[CPL];
  float mx = 0.0f;
#pragma unroll
  for (int p = 0; p < CPL / 8; ++p) {
    float x8[8];
    unpack8<BF16>(kraw[p], x8);
    const float4 m0 = mean4(c0 + 8 * p), m1 = mean4(c0 + 8 * p + 4);
    const float mean[8] = {m0.x, m0.y, m0.z, m0.w, m1.x, m1.y, m1.z, m1.w};
#pragma unroll
    for (int e = 0; e < 8; ++e) x[8 * p + e] = __fsub_rn(x8[e], mean[e]);
  }
  if (n0 + BKV > N) {                              // a block with padded keys: their codes and Delta-S are 0
#pragma unroll
    for (int e = 0; e < CPL; ++e) x[e] = n0 + r < N ? x[e] : 0.0f;
  }
  // A value that is not a number (a NaN key makes its channel's mean NaN, and so the channel of every key) leaves the scale alone and has
  // code 0, which the exact form of the codes gives and the FP6 conversion, that has no NaN, does not.  The maximum that passes NaN on takes
  // no instruction more than the one that does not.
  bool odd = false;
  if constexpr (INT4) {
#pragma unroll
    for (int e = 0; e < CPL; ++e) mx = __builtin_elementwise_maximum(mx, fabsf(x[e]));
    odd = __builtin_amdgcn_ballot_w64(mx != mx) != 0;
    if (odd) mx = 0.0f;
  }
  if (!INT4 || odd) {
#pragma unroll
    for (int e = 0; e < CPL; ++e) mx = fmaxf(mx, fabsf(x[e]));
  }
  // lanes l, l^16, l^32, l^48 hold one key: its maximum first, then (unless every key has its own
  // scale) the run of 4 keys, then (default) the wavefront's run of 16
  mx = butterfly_max<32>(butterfly_max<16>(mx));
  const float mx_key = mx;                         // this key's largest magnitude (DS_DIGITS: its fixed-point exponent)
  if (kg >= 4) mx = group_max<4>(mx);
  if (kg == 16) mx = butterfly_max<8>(butterfly_max<4>(mx));
  if (block_groups) {       // per-block granularity: one scale for the whole 64-key block
    if (lane == 0) s_bmax[w] = mx;
    __syncthreads();
    mx = fmaxf(fmaxf(s_bmax[0], s_bmax[1]), fmaxf(s_bmax[2], s_bmax[3]));
  }
  if (part == 0) {
  const float delta = head_scale ? head_scale[bhkv] : __fdiv_rn(mx, (float)QMAX);
  const int ksh = kg == 16 ? 4 : (kg == 4 ? 2 : 0);
  if (k4 == 0 && (r16 & (kg - 1)) == 0) k_scale[(bhkv * nKb + kb) * (BKV >> ksh) + ((16 * w + r16) >> ksh)] = delta;
  if (stats_only) return;                // per-tensor scales, first pass: only the block maxima are wanted
  uint8_t* img = reinterpret_cast<uint8_t*>(s_codes);
  CodeScale qs = code_scale(delta);
  qs.fast = qs.fast && !odd;
  if constexpr (INT4) {
    // the lane's CPL codes are CPL*6/32 consecutive dwords of one MFMA lane's payload (all 6 of
    // them when d = 128; dwords 0..2 or 3..5 when d = 64), or two whole payloads (d = 256)
    constexpr int NPL = CPL > 32 ? CPL / 32 : 1, CPP = CPL / NPL;
#pragma unroll
    for (int pl = 0; pl < NPL; ++pl) {
      Codes32 cd;
      if constexpr (CPP < 32) {
#pragma unroll
        for (int e = 0; e < 16; ++e) { cd.ev[e] = 0.0f; cd.od[e] = 0.0f; }
      }
      code_group<CPP, QMAX>(x + CPP * pl, delta, qs, [&](int e, float c) { cd.set(e, c); });
      const v6u pw = cd.pack();
      int lane_m, e0;
      const size_t op = k_op6(r, c0 + CPP * pl, D, &lane_m, &e0);
      const int d0 = (6 * e0) >> 5;
#pragma unroll
      for (int i = 0; i < CPP * 6 / 32; ++i)
        *reinterpret_cast<unsigned*>(img + op + op6_byte(lane_m, 4 * (d0 + i))) = pw[i];
    }
  } else {
#pragma unroll
    for (int i = 0; i < CPL / 16; ++i) {
      unsigned c[16];
      code_group_bytes<16, QMAX>(x + 16 * i, delta, qs, c);
      *reinterpret_cast<uint4*>(img + k_code_off(r, c0 + 16 * i, D)) = pack16(c);
    }
  }
  }
  if constexpr (INT4) store_q(0);
  __syncthreads();
  if (part == 0) {
    constexpr int BLK16 = (int)(k_block_bytes(D, INT4) / 16);
    uint4* dst = reinterpret_cast<uint4*>(k_codes + (bhkv * nKb + kb) * k_block_bytes(D, INT4));
#pragma unroll
    for (int i = t; i < BLK16; i += 256) dst[i] = s_codes[i];
  }

  if constexpr (INT4) {
    // the smoothed keys stay in FP32 registers and are widened per use (FP64 form): CPL more conversions per step instead
    // of 2 CPL more live registers
    const double kap = (double)kappa;
    const int qcol = c0 + (D >= 128 ? 16 * k4 : 0);
    // DS_DIGITS: the digits of this lane's CPL smoothed values as B operands of v_mfma_i32_16x16x64_i8.  An operand is
    // 16 bytes per lane; contraction slot (step st, lane group k4, byte j) is given channel CPL k4 + 16 st + j - any
    // assignment is valid as long as the A operand uses the same one.
    constexpr int NST = CPL / 16;
    v4i bd[DSD ? DS_ND : 1][DSD ? NST : 1];
    double key_up = 0.0;
    if constexpr (DSD) {
      const DsScale ks = ds_row_scale(mx_key);
      key_up = (double)ks.up * kap * 0x1p-64;      // 2^E of the key, times kappa; the accumulators are joined times 2^64
#pragma unroll
      for (int st = 0; st < NST; ++st) {
#pragma unroll
        for (int q4 = 0; q4 < 4; ++q4) {
          const float y[4] = {x[16 * st + 4 * q4], x[16 * st + 4 * q4 + 1], x[16 * st + 4 * q4 + 2], x[16 * st + 4 * q4 + 3]};
          unsigned dg[DS_ND];
          ds_digits4(y, ks.magic, dg);
#pragma unroll
          for (int a = 0; a < DS_ND; ++a) bd[a][st][q4] = (int)dg[a];
        }
      }
      // (opaque to the compiler from here on: it would otherwise form the digits anew in every step)
#pragma unroll
      for (int a = 0; a < DS_ND; ++a) {
#pragma unroll
        for (int st = 0; st < NST; ++st) asm volatile("" : "+v"(bd[a][st]));
      }
    }
    const unsigned rowstride = (unsigned)nKb * BKV;
    float* const out = delta_s + n0;
    for (int half = 0; step.R < row_end; half ^= 1) {
      // the next step's rows are on their way while this one is multiplied, and go to the other half of the buffer
      i += DS_ROWS;
      if (i >= nQs) { i -= nr; ++g; }
      const Step nxt = step_at(step.R + DS_ROWS, g, i);
      if (nxt.R < row_end) load_q(nxt);
      const int rows = min(nrow - step.R, DS_ROWS);
      const bool plain = plain_step(step);
      float* const out0 = out + (size_t)(unsigned)step.base * rowstride;      // (uniform: the lanes add 32-bit offsets)
      // the four values of a lane: rows rl + v rs of the step
      auto put4 = [&](int rl, int rs, const float (&val)[4]) {
        if (plain) {
          const unsigned off = (unsigned)rl * rowstride + (unsigned)r;
#pragma unroll
          for (int v = 0; v < 4; ++v) (out0 + (size_t)(unsigned)(v * rs) * rowstride)[off] = val[v];
        } else {
#pragma unroll
          for (int v = 0; v < 4; ++v) {
            int rr = rl + v * rs;
            asm volatile("" : "+v"(rr));
            const int row = step_row(step, rr);
            if (row >= 0) out[(size_t)(unsigned)row * rowstride + (unsigned)r] = val[v];
          }
        }
      };
      float val[4] = {0.0f, 0.0f, 0.0f, 0.0f};
      if (zero_ds) {                               // (Q not smoothed: the block means are zero and so is Delta-S)
        put4(4 * k4, 1, val);
      } else if constexpr (DSD) {
        // accumulators by digit-pair weight: acc[k] collects the pairs with a + b = k; result element v of lane l is
        // row 4 (l / 16) + v, column l % 16
        v4i acc[DS_MAXPAIR + 1];
#pragma unroll
        for (int a = 0; a < DS_ND; ++a) {
#pragma unroll
          for (int st = 0; st < NST; ++st) {
            const v4i qa = *reinterpret_cast<const v4i*>(&s_qd[half * DS_ROWS + r16][a * D + CPL * k4 + 16 * st]);
#pragma unroll
            for (int b = 0; b < DS_ND && a + b <= DS_MAXPAIR; ++b) {
              // the first pair of a weight starts from zero (a constant operand of the instruction)
              const bool first = st == 0 && a == (a + b >= DS_ND ? a + b - (DS_ND - 1) : 0);
              acc[a + b] = __builtin_amdgcn_mfma_i32_16x16x64_i8(qa, bd[b][st], first ? v4i{0, 0, 0, 0} : acc[a + b], 0, 0, 0);
            }
          }
        }
#pragma unroll
        for (int v = 0; v < 4; ++v) {
          // 2^64 sum_k acc_k 2^(-8 (k + 2)): neighbours joined as integers first, then float64, smallest weights first.
          // 256 acc_k + acc_{k+1} < 2^31 at d = 128: the largest is k = 4, where the five pairs of digits come to at
          // most 3.5 2^14 per channel - a number has 24 consecutive significant bits, so that one with n_0 beyond a carry has
          // n_4 = 0.  At d = 256 that bound does not hold, and all of them are joined in float64.
          static_assert(DS_ND == 6 && DS_MAXPAIR == 6, "seven accumulators");
          double sum = (double)acc[6][v];
          if constexpr (D <= 128) {
            const int u0 = acc[0][v] * 256 + acc[1][v], u1 = acc[2][v] * 256 + acc[3][v], u2 = acc[4][v] * 256 + acc[5][v];
            sum = __fma_rn((double)u2, 0x1p8, sum);
            sum = __fma_rn((double)u1, 0x1p24, sum);
            sum = __fma_rn((double)u0, 0x1p40, sum);
          } else {
            sum = __fma_rn((double)acc[5][v], 0x1p8, sum);
            sum = __fma_rn((double)acc[4][v], 0x1p16, sum);
            sum = __fma_rn((double)acc[3][v], 0x1p24, sum);
            sum = __fma_rn((double)acc[2][v], 0x1p32, sum);
            sum = __fma_rn((double)acc[1][v], 0x1p40, sum);
            sum = __fma_rn((double)acc[0][v], 0x1p48, sum);
          }
          val[v] = (float)(sum * (s_qs[half * DS_ROWS + 4 * k4 + v] * key_up));
        }
        put4(4 * k4, 1, val);
      } else if constexpr (DS32) {
        // Faster, approximate form (an option of the boundary): the same product on the FP32 form of the
        // instruction (result element v of lane l is row 4*(l/16) + v, column l%16).  FP32 accumulation:
        // within (d + 2) 2^-24 kappa sum_c |q_bar_c gamma(K)_c| of the exact value, about half a unit of 2^-24 of
        // that magnitude on average.  It runs at twice the rate and under the vector work of the workgroups
        // that share the CU, so the product costs next to nothing on top of the quantization.
        v4f acc = {0.0f, 0.0f, 0.0f, 0.0f};
#pragma unroll
        for (int cs = 0; cs < CPL; ++cs)
          acc = __builtin_amdgcn_mfma_f32_16x16x4f32(s_q[half * DS_ROWS + r16][qcol + cs], x[cs], acc, 0, 0, 0);
#pragma unroll
        for (int v = 0; v < 4; ++v) val[v] = __fmul_rn(kappa, acc[v]);
        put4(4 * k4, 1, val);
      } else if (rows <= 8) {
        // A few rows: four at a time by v_mfma_f64_4x4x4_4b_f64, four independent 4 x 4 products per instruction (lane l supplies
        // A[l % 4][l / 16] and B[l / 16][l % 4] of product (l / 4) % 4 and receives D[l / 16][l % 4]): 18 cycles for the step of
        // four channels that takes the 16-row form 64, and the same order of additions.
#pragma unroll 1
        for (int r4 = 0; r4 < rows; r4 += 4) {
          double acc = 0.0;
#pragma unroll
          for (int cs = 0; cs < CPL; ++cs) {
            asm volatile("" : "+v"(x[cs]));        // keeps the widening where it is used
            acc = __builtin_amdgcn_mfma_f64_4x4x4f64((double)s_q[half * DS_ROWS + r4 + (r16 & 3)][qcol + cs], (double)x[cs], acc, 0, 0, 0);
          }
          const int row = step_row(step, r4 + k4);
          if (row >= 0) out[(size_t)(unsigned)row * rowstride + (unsigned)r] = (float)(kap * acc);
        }
      } else {
        // FP64 MFMA lane map: lane l supplies A[l%16][l/16] and B[l/16][l%16]; result element v of lane l is row
        // 4*v + l/16, column l%16
        v4d acc = {0.0, 0.0, 0.0, 0.0};
#pragma unroll
        for (int cs = 0; cs < CPL; ++cs) {
          asm volatile("" : "+v"(x[cs]));          // keeps the widening inside the loop
          acc = __builtin_amdgcn_mfma_f64_16x16x4f64((double)s_q[half * DS_ROWS + r16][qcol + cs], (double)x[cs], acc, 0, 0, 0);
        }
#pragma unroll
        for (int v = 0; v < 4; ++v) val[v] = (float)(kap * acc[v]);
        put4(k4, 4, val);
      }
      if (nxt.R >= row_end) break;
      store_q(half ^ 1);                           // (its last readers met the barrier that opened this step)
      __syncthreads();
      step = nxt;
    }
  }
}

// ------------------------------------------------------------------------------------------
// V: per-channel FP8 codes (E4M3, or E5M2 with the E5M2 template flag), transposed into the A-operand
// order of the P~V product
// (Sec. 3.3; Algorithm 1 "Preprocessing": (delta_V, V^) = psi_V(V)).  v_mean is null, or the token
// mean to subtract first (smooth-V option, SMOOTH_V).
// One workgroup per 64 keys of one (batch, KV head); a thread owns VCH channels of four (d = 256: eight) consecutive keys.
// The conversion instruction takes its pair of values from two keys of a channel, so that a result word is four keys of
// one channel - the transposition costs nothing but where the word goes in the LDS image of the block, which then
// leaves in 16-byte pieces.  The rows are requested before the scales (or the partial maxima they come from) and all together,
// and the quotients are three instructions instead of a division.  Bound: the loads (202 MB for 128 heads of 4096 tokens).
// Against a byte at a time out of LDS, a division per value and a row per round trip, the whole preprocessing: 128 heads of
// 1024 tokens 58.7 -> 55.6 us, 32 of 8192, 8-bit mode, 91.2 -> 88.1, 16 of 8192 of 256 channels 132.9 -> 128.4, 96 of 17776 of
// 64 channels 700 -> 685, 128 of 4096 202.2 -> 200.4.  E5M2 and INT8 keep the division, and so does a head of E4M3 with a channel of zeros
// (64 of 4096, 16 of 8192, 32 of 600 tokens, all widths: 0.96 to 1.00 of the form before for those two, 0.95 to 1.00 with one such channel).
template <int D, bool REDUCE> struct QuantVLds {
  uint4 img[BKV * D / 16];                         // the block's packed codes, piece i at v_piece(i)
  float vscale[REDUCE ? D : 1];                    // delta_V of this head, reduced here
};
// Where piece i of a block's codes sits in LDS: its channel is i % 32 of tile i / 128, and the 16 threads that write side by
// side own every VCH-th channel - spread over the low bits they meet in no bank.
__device__ __forceinline__ int v_piece(int i) { return i ^ (((i >> 4) & 1) | ((i >> 6) & 6)); }
template <bool BF16, int D, bool SMOOTH_V, int PVF, bool REDUCE = false>
__device__ __forceinline__ void quant_v_block(QuantVLds<D, REDUCE>& lds, const BlockPos bp, const QuantKV& a) {
  const unsigned short* __restrict__ V = a.v;
  const float* __restrict__ v_mean = a.v_mean; uint8_t* __restrict__ v_codes = a.v_codes;
  const int Nq = a.Nq, Nmax = a.Nk, nKb = a.nKb;
  const TensorMap& km = a.km; const SeqMap& sm = a.sm;
  constexpr int VCH = D == 64 ? 4 : 8, NCG = D / VCH, NRG = 256 / NCG, RPT = BKV / NRG;
  static_assert(RPT % 4 == 0, "whole words of four keys");
  auto& s_vscale = lds.vscale;
  const int t = threadIdx.x, cg = t % NCG, rg = t / NCG;
  const int kb = bp.x;
  const size_t bh = bp.y;
  const int n0 = kb * BKV;
  const HeadPos hp = head_pos(km, bp.y);
  const Seq sq = seq_of(sm, hp.b, Nq, Nmax);
  const int N = sq.nk;
  if (n0 >= N) return;                             // a block past the end of a shorter sequence
  const size_t hbase = hp.base + sq.k0 * (size_t)km.sn;
  // every row is requested before anything else of the block (rows past the end read the last one; their codes are 0)
  unsigned raw[RPT][VCH / 2];
#pragma unroll
  for (int i = 0; i < RPT; ++i) {
    const unsigned short* src = V + row_offset(km, hbase, min(n0 + rg * RPT + i, N - 1)) + cg * VCH;
    if constexpr (VCH == 8) {
      const uint4 r = nt_load16(src);
      raw[i][0] = r.x; raw[i][1] = r.y; raw[i][2] = r.z; raw[i][3] = r.w;
    } else {
      const uint2 r = nt_load8(src);
      raw[i][0] = r.x; raw[i][1] = r.y;
    }
  }
  if constexpr (REDUCE) {
    if (t < D) {
      float vm = 0.0f;
      for (int ch = 0; ch < a.nchunk; ch += SUM_BATCH) {
        float x[SUM_BATCH];
#pragma unroll
        for (int i = 0; i < SUM_BATCH; ++i) x[i] = __uint_as_float(a.v_max[(bh * a.nchunk + min(ch + i, a.nchunk - 1)) * D + t]);
#pragma unroll
        for (int i = 0; i < SUM_BATCH; ++i) vm = fmaxf(vm, x[i]);
      }
      const float v = __fdiv_rn(vm, a.code_max);
      s_vscale[t] = v;
      if (kb == 0) a.v_scale[bh * D + t] = v;
    }
    __syncthreads();
  }
  float sc[VCH], rc[VCH], mean[VCH];
  bool fast = PVF == PV_E4M3;
#pragma unroll
  for (int e = 0; e < VCH; ++e) {
    sc[e] = REDUCE ? s_vscale[cg * VCH + e] : a.v_scale[bh * D + cg * VCH + e];
    mean[e] = SMOOTH_V ? v_mean[bh * D + cg * VCH + e] : 0.0f;
    fast = fast && div_by_ok(sc[e]);
  }
  fast = __builtin_amdgcn_ballot_w64(!fast) == 0;
#pragma unroll
  for (int e = 0; e < VCH; ++e) rc[e] = fast ? __fdiv_rn(1.0f, sc[e]) : 0.0f;
  uint8_t* img = reinterpret_cast<uint8_t*>(lds.img);
  const bool ragged = n0 + BKV > N;
  // The quotient: div_by; with a supplied scale, which bounds nothing, div_by with its remainder kept finite, since an infinite quotient has none
  // (the conversion tells infinities from NaN); or a division, also where a scale taken from the values is infinite.
  enum { BOUNDED, UNBOUNDED, EXACT };
  auto convert = [&](auto form) {
    constexpr int FORM = decltype(form)::value;
#pragma unroll
    for (int k = 0; k < RPT / 4; ++k) {
      const int key0 = rg * RPT + 4 * k;
#pragma unroll
      for (int e = 0; e < VCH; ++e) {
        float x[4];
#pragma unroll
        for (int i = 0; i < 4; ++i) {
          const unsigned w = raw[4 * k + i][e >> 1];
          x[i] = load16<BF16>((unsigned short)((e & 1) ? w >> 16 : w & 0xffffu));
          if constexpr (SMOOTH_V) x[i] = __fsub_rn(x[i], mean[e]);
        }
        if (ragged) {
#pragma unroll
          for (int i = 0; i < 4; ++i) x[i] = n0 + key0 + i < N ? x[i] : 0.0f;
        }
        if constexpr (FORM != EXACT) {
          // div_by with the remainder's sign turned, so that a quotient of -0 stays -0
#pragma unroll
          for (int i = 0; i < 4; ++i) {
            const float q = __fmul_rn(x[i], rc[e]);
            float rem = __fmaf_rn(q, sc[e], -x[i]);
            if constexpr (FORM == UNBOUNDED) rem = __builtin_amdgcn_fmed3f(rem, -0x1.fffffep127f, 0x1.fffffep127f);
            x[i] = __fmaf_rn(rem, -rc[e], q);
          }
        } else {
#pragma unroll
          for (int i = 0; i < 4; ++i) {
            x[i] = sc[e] > 0.0f ? __fdiv_rn(x[i], sc[e]) : 0.0f;
            asm volatile("" : "+v"(x[i]) :: "memory");     // (one division at a time)
          }
        }
        int wd = 0;
        if constexpr (PVF == PV_INT8) {
          // psi of Sec. 2.2 with qmax 127: |x / delta_V| <= 127 (1 + 2^-23), round-half-even, two's-complement bytes
#pragma unroll
          for (int i = 0; i < 4; ++i) wd |= ((int)rintf(x[i]) & 0xff) << (8 * i);
        } else if constexpr (PVF == PV_E5M2) {
          wd = __builtin_amdgcn_cvt_pk_bf8_f32(x[0], x[1], wd, false);
          wd = __builtin_amdgcn_cvt_pk_bf8_f32(x[2], x[3], wd, true);
        } else {
          wd = __builtin_amdgcn_cvt_pk_fp8_f32(x[0], x[1], wd, false);
          wd = __builtin_amdgcn_cvt_pk_fp8_f32(x[2], x[3], wd, true);
        }
        const int off = (int)v_code_off(key0, cg * VCH + e, D);
        *reinterpret_cast<int*>(img + 16 * v_piece(off >> 4) + (off & 15)) = wd;
      }
    }
  };
  if (!fast) convert(std::integral_constant<int, EXACT>{});
  else if (REDUCE || a.bounded) convert(std::integral_constant<int, BOUNDED>{});
  else if constexpr (!REDUCE) convert(std::integral_constant<int, UNBOUNDED>{});
  __syncthreads();
  uint4* dst = reinterpret_cast<uint4*>(v_codes + (bh * nKb + kb) * (size_t)BKV * D);
  for (int i = t; i < BKV * D / 16; i += 256) dst[i] = lds.img[v_piece(i)];
}

// Workgroups per CU the K quantizer is built for.  Digits: the six digit planes of a lane's channels and the seven accumulators
// stay in registers through the steps, 124 registers of 128 at d = 128 (4096 tokens of 128 heads: three workgroups per CU 97 us,
// four 91; as long as the loads of a step across heads kept their addresses through the loop, seven registers spilled once per
// workgroup, 58 MB), 96 at d = 64 (four 467 us of a 17776-token call, five 435); d = 256 fits two.
template <int D, bool INT4, int DSM> constexpr int quant_k_occupancy() { return D == 256 ? 2 : (D == 64 && INT4 && DSM == DS_DIGITS ? 5 : 4); }
template <bool BF16, bool INT4, int D, int DSM = DS_DIGITS>
__global__ void __launch_bounds__(256, (quant_k_occupancy<D, INT4, DSM>())) k_quant_k(const QuantKV a) {
  __shared__ QuantKLds<D, INT4, DSM, false> lds;
  quant_k_block<BF16, INT4, D, DSM>(lds, block_pos(a.km), a, (int)blockIdx.z);
}
template <bool BF16, int D, bool SMOOTH_V, int PVF>
__global__ void __launch_bounds__(256) k_quant_v(const QuantKV a) {
  __shared__ QuantVLds<D, false> lds;
  quant_v_block<BF16, D, SMOOTH_V, PVF>(lds, block_pos(a.km), a);
}

// ------------------------------------------------------------------------------------------
// Small calls: a launch that fills a fraction of the chip costs its latency (3 to 7 us) whatever it does, so the six
// launches of the general sequence become three: Q and the statistics side by side, then K and V side by side with
// the reduction of the statistics in front (each workgroup for its own head), then the attention kernel.
// Where a kernel of the sequence fills the chip by itself the pair is slower than the two (the workgroups of one
// take the slots and registers of the other): see the rule, small_call.
struct SmallStats {
  const unsigned short *k, *v;
  double* k_sum;
  unsigned* v_max;
  int nchunk;
  TensorMap km;
  int turn_shift, turn_mask;
  float inv_nQb;
};
template <bool BF16, bool INT4, int D>
__global__ void __launch_bounds__(256, D == 256 || !INT4 ? 2 : 4) k_quant_q_and_stats(const QuantQ q, const SmallStats st) {
  __shared__ Overlay<QuantQLds<D, INT4>, StatsLds<D, false>> lds;
  // A row of the grid: the query blocks of a KV head's heads, then its chunks.  Workgroups go to the eight XCDs in turn, so that in rows of an
  // even length the query blocks would fall on some of them only: a row that begins where an earlier one did is turned.  (On a grid of
  // (query blocks and chunks, heads), the places of the grouped heads' chunks empty, 39 x 64 heads on 8 of 58 queries and 586 keys, 256
  // channels, 8-bit took 378 us, turned 133; the whole call 598, now 353, six launches 370.  All query blocks in front of all chunks: 128
  // heads of 1024 tokens 23.4, here 21.6; 44 x 64 on 16 of 158 queries and 316 keys, 64 channels, 8-bit 51.3, here 40.9.)
  const unsigned nQb = (unsigned)q.nQb, nq = nQb * (unsigned)q.G;
  unsigned x = blockIdx.x + ((blockIdx.y >> st.turn_shift) & (unsigned)st.turn_mask);
  if (x >= gridDim.x) x -= gridDim.x;
  if (x < nq) {
    // x / nQb: (x + 1/2) / nQb is at least 1 / (2 nQb) from an integer, and the error of its FP32 value below 2^-22 x / nQb
    const unsigned g = q.G == 1 ? 0u : (unsigned)__builtin_amdgcn_readfirstlane((int)(((float)x + 0.5f) * st.inv_nQb));
    quant_q_block<BF16, INT4, D>(lds.a, q_block(q, x - g * nQb, blockIdx.y * (unsigned)q.G + g), q);
  } else {
    col_stats_block<BF16, D, false>(lds.b, BlockPos{x - nq, blockIdx.y, (unsigned)st.nchunk}, st.k, st.v, st.k_sum, nullptr, st.v_max, q.N, q.Nk,
                                    st.km, q.sm);
  }
}
// K and V of a key block side by side, so that the one's arithmetic runs under the other's loads and stores whatever the length.
template <bool BF16, bool INT4, int D, int DSM, bool SMOOTH_V, bool REDUCE>
__global__ void __launch_bounds__(256, (quant_k_occupancy<D, INT4, DSM>())) k_quant_kv(const QuantKV a) {
  __shared__ Overlay<QuantKLds<D, INT4, DSM, REDUCE>, QuantVLds<D, REDUCE>> lds;
  BlockPos bp = block_pos(a.km);
  const bool is_v = a.mixed ? pair_second(blockIdx.y * gridDim.x + blockIdx.x) : (bp.x & 1) != 0;
  bp.x >>= 1; bp.nx >>= 1;
  if (!is_v) quant_k_block<BF16, INT4, D, DSM, REDUCE>(lds.a, bp, a, (int)blockIdx.z);
  else if (blockIdx.z == 0) quant_v_block<BF16, D, SMOOTH_V, PV_E4M3, REDUCE>(lds.b, bp, a);
}

// ------------------------------------------------------------------------------------------
// Per-tensor scales (the coarsest granularity of the paper's comparison, Sec. 2.2): the quantizers run
// once in per-block mode just to leave every block's scale, this kernel takes the largest scale of a
// head (delta = fl32(max / qmax) is monotone in the maximum, so the largest block scale is the
// head's), and the quantizers run again with that scale.  One workgroup per head; `per_block` scale
// entries per block, `stride` entries per head, blocks counted from the sequence's own length.
__global__ void __launch_bounds__(256) k_head_scale(const float* __restrict__ scale, float* __restrict__ head_scale,
                                                    int per_block, int stride, int tokens_per_block, int heads,
                                                    int which_k, int Nq, int Nk, SeqMap sm) {
  __shared__ float s_m[4];
  const unsigned head = blockIdx.x;
  const Seq sq = seq_of(sm, head / (unsigned)heads, Nq, Nk);
  const int n = which_k ? sq.nk : sq.n;
  const int entries = ((n + tokens_per_block - 1) / tokens_per_block) * per_block;
  float m = 0.0f;
  for (int i = threadIdx.x; i < entries; i += 256) m = fmaxf(m, scale[(size_t)head * stride + i]);
  m = wave_max(m);
  if ((threadIdx.x & 63) == 0) s_m[threadIdx.x >> 6] = m;
  __syncthreads();
  if (threadIdx.x == 0) head_scale[head] = fmaxf(fmaxf(s_m[0], s_m[1]), fmaxf(s_m[2], s_m[3]));
}

// ------------------------------------------------------------------------------------------
// Copies from the packed workspace to plain layouts (used only by sage_attn_quant).
__global__ void k_unpack_codes(const int8_t* __restrict__ packed, int8_t* __restrict__ plain, int N,
                               int d, size_t slab, int which, int fp6) {
  // grid: (ceil(N*d/256), heads); which: 0 = q, 1 = k, 2 = v; fp6: q/k hold 6-bit E2M3 codes
  const size_t i = (size_t)blockIdx.x * blockDim.x + threadIdx.x;
  if (i >= (size_t)N * d) return;
  const int n = (int)(i / d), c = (int)(i % d);
  const uint8_t* src = reinterpret_cast<const uint8_t*>(packed) + (size_t)blockIdx.y * slab;
  int8_t b;
  if (fp6 && which != 2) {
    int lane_m, e;
    const size_t op = which == 0 ? q_op6(n, c, d, &lane_m, &e) : k_op6(n, c, d, &lane_m, &e);
    const int bit = 6 * e, by = bit >> 3;
    unsigned v = src[op + op6_byte(lane_m, by)];
    if (by + 1 < 24) v |= (unsigned)src[op + op6_byte(lane_m, by + 1)] << 8;
    b = (int8_t)e2m3_to_int4_code((v >> (bit & 7)) & 63u);
  } else {
    const size_t off = which == 0 ? q_code_off(n, c, d) : (which == 1 ? k_code_off(n, c, d) : v_code_off(n, c, d));
    b = (int8_t)src[off];
  }
  plain[(size_t)blockIdx.y * N * d + i] = b;
}

__global__ void k_unpack_rows(const float* __restrict__ src, float* __restrict__ dst, int n_valid,
                              int src_stride) {
  // grid: (ceil(n_valid/256), rows): dst[row][0..n_valid) = src[row][0..n_valid)
  const int i = blockIdx.x * blockDim.x + threadIdx.x;
  if (i < n_valid) dst[(size_t)blockIdx.y * n_valid + i] = src[(size_t)blockIdx.y * src_stride + i];
}

// ------------------------------------------------------------------------------------------
// The statistics pass: mean(K) and delta_V (and mean(V) with the smooth-V option) into P.k_mean, P.v_scale, P.v_mean.
static Finalize finalize_args(const Dims& Dm, const Ptrs& P) {
  return {P.k_sum, Dm.smooth_v ? P.v_sum : nullptr, P.v_max, P.k_mean, P.v_mean, P.v_scale, Dm.B * Dm.Hkv * Dm.d, Dm.N, Dm.Nk, Dm.d, Dm.Hkv,
          (Dm.Nk + STAT_ROWS - 1) / STAT_ROWS, Dm.seq, Dm.pvf == PV_INT8 ? INT8_PV_MAX : (Dm.pvf == PV_E5M2 ? E5M2_MAX : E4M3_MAX), Dm.smooth_k};
}
// finalize = false: the caller's next launch does it (no smooth_v)
template <bool BF16, int D>
static void launch_stats_t(const Dims& Dm, const Ptrs& P, hipStream_t s, bool finalize = true) {
  const unsigned short* k = (const unsigned short*)P.k;
  const unsigned short* v = (const unsigned short*)P.v;
  const TensorMap km = make_tensor_map(Dm.nhd, Dm.Hkv, Dm.Nk, Dm.d, Dm.seq.cu_q != nullptr);
  const Finalize f = finalize_args(Dm, P);
  const dim3 gstat = block_grid(km, f.nchunk, Dm.B * Dm.Hkv);
  const int fin = (f.n + FIN_ENT - 1) / FIN_ENT;
  if (Dm.smooth_v) k_col_stats<BF16, D, true><<<gstat, 256, 0, s>>>(k, v, P.k_sum, P.v_sum, P.v_max, Dm.N, Dm.Nk, km, Dm.seq);
  else k_col_stats<BF16, D, false><<<gstat, 256, 0, s>>>(k, v, P.k_sum, nullptr, P.v_max, Dm.N, Dm.Nk, km, Dm.seq);
  if (finalize) k_finalize_stats<<<fin, FIN_ENT * FIN_PARTS, 0, s>>>(f);
  if (Dm.smooth_v) {
    k_v_absmax<BF16, D><<<gstat, 256, 0, s>>>(v, P.v_mean, P.v_max, Dm.N, Dm.Nk, km, Dm.seq);
    k_finalize_vscale<<<fin, FIN_ENT * FIN_PARTS, 0, s>>>(P.v_max, P.v_scale, f.n, Dm.d, f.nchunk, f.code_max);
  }
}

// Calls that the three-launch sequence serves (k_quant_q_and_stats, k_quant_kv): E4M3, exact Delta-S, no row constants (they need mean(K)
// before Q).  What it costs is the reduction of the statistics, which every workgroup does for its head: the workgroups of the general
// sequence's Q and K launches times the chunks of a head.  Whole calls, full attention, us, general sequence (K and V as kv_pair says) /
// three launches, 4-bit then 8-bit: 2 heads of 64 channels, 256 tokens 19.1 / 15.9, 19.6 / 16.3; 128 of 128, 500 tokens (1536 workgroups, 2
// chunks) 62.6 / 51.0, 61.8 / 53.9; 512 of 200 (3072, 1) 83.6 / 75.1, 81.8 / 71.7; 128 of 1024 (3072, 4) 115.3 / 113.8, 117.3 / 112.5; 32
// on 8 of 3000 (1144, 12) 137.5 / 134.1, 146.4 / 143.1; 8 of 5000 (952, 20) 151.4 / 149.5, 150.0 / 148.0; 8 on 1 of 8000 (629, 32) 232.3 /
// 233.5, 212.5 / 211.8; 2 of 12000 (564, 47) 162.3 / 165.9, 164.8 / 171.5; 32 on 8 of 3362 (1288, 14), 4-bit, causal 113.3 / 106.6.  By workgroups
// times chunks, general / three: 4-bit 10000 to 14336, 64 channels 1.00 to 1.03, 128 1.01 to 1.04, 15000 to 20480 0.99 to 1.01, 0.96 (many
// key blocks) to 1.06 (many rows of block means); 8-bit 15000 to 20480 0.99 to 1.09; 21000 to 40000 0.92 to 1.02.
// The bodies of a pair share its LDS (side by side it held pairs of d >= 128 to fewer workgroups), but its registers are the larger body's,
// which tells in the 4-bit mode at 256 channels where the chip is full: it gains to 768 key blocks, with many rows of block means to 384
// (64 on 8 heads of 1607 queries and 3214 keys, 408 blocks, 104 rows, statistics supplied 317 / 325; 64 heads of 750 tokens 103.2 / 99.2,
// 64 of 1000 with 1024 blocks 121.7 / 123.9, 256 of 512 with 2048 183 / 194; 8-bit 99.1 / 88.2, 121.5 / 112.0, 190 / 174).
constexpr int SMALL_CALL_WORK = 20480, SMALL_CALL_CHUNKS = 32;
// Rows of block means that a key block meets: up to 24, two steps of the Delta-S product, K's workgroups are about as long as V's.
static bool few_rows(const Dims& Dm) { return (long long)(Dm.H / Dm.Hkv) * Dm.nQb <= 24; }
bool small_call(const Dims& Dm) {
  const long long nk = (long long)Dm.B * Dm.Hkv * Dm.nKb, nq = (long long)Dm.B * Dm.H * Dm.nQb;
  const int nchunk = (Dm.Nk + STAT_ROWS - 1) / STAT_ROWS;
  if (Dm.d == 256 && Dm.int4 && nk > (few_rows(Dm) ? 768 : 384)) return false;
  return !Dm.want_lse && !Dm.smooth_v && !Dm.tensor_groups && Dm.pvf == PV_E4M3 && !Dm.ds32 && !Dm.seq.cu_q &&
         nchunk <= SMALL_CALL_CHUNKS && (nk + nq) * nchunk <= SMALL_CALL_WORK;
}

// K and V in one launch (k_quant_kv) for larger calls too: the one's loads and stores run under the other's arithmetic, and one launch
// and one tail are saved.  The registers are the larger body's, K's with Delta-S, so where K fills the chip by itself and its workgroups are
// long (many rows of block means) V's are better off in a launch of their own.  A packed batch is counted by its longest sequence, which is all
// that is known here; the lines hold for it as they do for a batch of fixed length.
// 4-bit mode, 64 and 128 channels, preprocessing alone on inputs in turn, one launch over two, some 1400 calls of both kinds and layouts by key
// blocks and rows per KV head, lowest to highest (mean): up to 800 blocks 0.84 to 1.03 (0.92; 250 to 2200 rows 0.91 to 1.01).  Up to 24
// rows, 801 to 4608 blocks 0.86 to 1.02 (0.96), 4609 to 7000 of 64 channels 0.94 to 1.00 (0.98), of 128 0.98 to 1.04 (1.00), more of 64
// channels 0.92 to 1.07 (1.00), of 128 0.96 to 1.08 (1.03).  More rows by their product with the blocks: 25 to 256 rows, up to 393216 0.88 to 1.02 (0.97), to 600000 0.90 to 1.05 (0.99), to
// 900000 0.96 to 1.03 (1.00), more 0.97 to 1.09 (1.02); more than 256 rows and 800 blocks 0.92 to 1.12 (1.00).
// 256 channels, whole calls, time of two launches / one: 250, 39 rows 1.04, 328 to 432, 48 to 72 rows 0.99, 500, 56 rows 0.97,
// 512 to 640, 1 to 24 rows 1.00 to 1.04, 736, 12 rows 0.99, 960, 2 rows 0.95.  8-bit, whose two quantizers are alike, 64 and 128 channels,
// us: 1536 blocks 119.3 / 118.2, 3912 142.5 / 140.6, 4928 165.8 / 165.0, 5056 139.4 / 140.9, 7360 315.3 / 320.0, 13496 234.4 / 238.3; 256
// channels 584 179.4 / 176.4, 768 74.9 / 74.2, 2048 389 / 409.
static bool kv_pair(const Dims& Dm) {
  if (Dm.tensor_groups || Dm.pvf != PV_E4M3 || Dm.ds32) return false;
  const long long blocks = (long long)Dm.B * Dm.Hkv * Dm.nKb, rows = (long long)(Dm.H / Dm.Hkv) * Dm.nQb;
  if (Dm.d == 256) return blocks <= (!Dm.int4 || Dm.seq.cu_q ? 768 : few_rows(Dm) ? 640 : 320);
  if (!Dm.int4 || few_rows(Dm)) return blocks <= 4608;
  return blocks <= 800 || (rows <= 256 && blocks * rows <= 600000);
}

// Workgroups per key block of K, each with its share of the steps of the Delta-S product (and the loads and digits of the keys once more): where
// the key blocks are few and the block means many - grouped KV heads, a long sequence - a workgroup per key block leaves much of the chip idle for
// the length of its chain.  Steps are counted for the blocks that see all rows: under a causal mask later ones have fewer, to none.
// 64 and 128 channels, of which four workgroups fit a CU: three rounds of those, divided by the key blocks and rounded up - two parts up to just
// under three rounds of key blocks, six of workgroups - with four steps each, or six where the key blocks alone make half a round.
// Preprocessing, us, one / as many: 8 on 1 heads of 25318 tokens (396 key blocks, 99 steps) 157.8 /
// 96.5, without a mask 167 / 130, 16 on 2 of 6000 56.3 / 36.9, 8 on 1 of 12000 of 64 channels 62.0 / 30.7, 48 on 6 of 4000 of 64 43.0 / 34.3, 4 on 2
// of 32965 (1032, 33 steps) 95.5 / 86.3, 32 on 8 of 16384 (2048, 32) 169.4 / 165.2, 96 on 12 of 12000 (2256, 47) 284.6 / 275.1, 56 on 7 of 25000 (2737, 98) 515 /
// 489; but 2 of 20000 (626, 10 steps) two 39.5 for 38.8, 4 of 16384 (1024, 8 steps) 48.7 for 48.5.  Rounded up over rounded down, 158 shapes between: two parts
// for one 0.89 to 1.02 (mean 0.96), three or four for one less 0.95 to 1.03 (1.00).
// 256 channels, where cutting the keys takes longer and one workgroup uses a CU nearly as well as the two that fit: without a mask all chains are equal, and
// parts gain where they level the CUs out, not where 256, 512 or 1000 workgroups already do (one / as the other widths, 64 on 4 of 4000 tokens, 252 blocks
// of 32 steps, the kernel 85 / 102; preprocessing of 4 on 1 of 16000 117 / 135, 16 on 2 of 8000 133 / 149, but 125 blocks of 32 steps two 74 for 93, 375 of 63 four
// 224 for 254, 750 of 63 two 345 for 358).  Under a mask they level the chains: 250 blocks of 63 steps 165 / 136 with two, 150 with seven, 125 of 32 91.5 / 66
// with three, 73 with eight; long sequences of one or two heads need the steps (938 blocks of 15 two 100 for 93).  136 shapes without a mask, as many over one: 0.59
// to 1.02, mean 0.95, and 166 with one 0.48 to 1.04, 0.92; by the rule of the other widths 0.97, to 1.16, and 0.92, to 1.09.  Packed batches, which have
// fewer blocks than their longest sequence lets one count, by the rule of the other widths (60 under a mask 0.60 to 1.05, mean 0.90, 60 without 0.71 to 1.05,
// 0.93; two parts for all of more than 128 blocks alike on average, with up to 16 % lost on two or three sequences).
static int k_parts(const Dims& Dm) {
  if (!Dm.int4 || Dm.ds_mode != DS_DIGITS || Dm.tensor_groups || !Dm.smooth_q) return 1;
  const long long blocks = (long long)Dm.B * Dm.Hkv * Dm.nKb, steps = ((long long)(Dm.H / Dm.Hkv) * Dm.nQb + DS_ROWS - 1) / DS_ROWS;
  const long long slots = Dm.d == 256 ? 512 : 1024;
  long long parts, each;                 // at most so many, with so many steps
  if (Dm.d < 256 || Dm.seq.cu_q) { parts = (3 * slots + blocks - 1) / blocks; each = 2 * blocks < slots ? 4 : 6; }
  else if (blocks <= 128) { parts = (Dm.causal ? 384 : 256) / blocks; each = 4; }
  else if (Dm.causal) {
    parts = blocks <= 256 ? 2 : (3 * slots + blocks - 1) / blocks;
    each = blocks <= 200 ? 4 : (blocks <= 256 ? 6 : (blocks <= 768 ? 8 : 12));
  } else if (blocks <= 256) { parts = blocks <= 170 ? 3 : (blocks <= 200 ? 2 : 1); each = 4; }
  else if (blocks <= 640) { parts = (blocks - 1) % 256 >= 128 ? 1 : (steps >= 48 ? 4 : 2); each = 6; }
  else { parts = blocks < 1536 ? 2 : 1; each = 12; }
  return (int)max(1LL, min(min(parts, steps / each), 8LL));
}

template <bool BF16, bool INT4, int D>
static hipError_t launch_prologue_t(const Dims& Dm, const Ptrs& P, hipStream_t s) {
  const int BH = Dm.B * Dm.H, BHkv = Dm.B * Dm.Hkv;
  const unsigned short* q = (const unsigned short*)P.q;
  const unsigned short* k = (const unsigned short*)P.k;
  const unsigned short* v = (const unsigned short*)P.v;
  const bool varlen = Dm.seq.cu_q != nullptr;
  const TensorMap qm = make_tensor_map(Dm.nhd, Dm.H, Dm.N, Dm.d, varlen),
                  km = make_tensor_map(Dm.nhd, Dm.Hkv, Dm.Nk, Dm.d, varlen);
  const SeqMap sm = Dm.seq;
  const float* v_mean = Dm.smooth_v ? P.v_mean : nullptr;
  QuantQ qa;
  qa.q = q; qa.q_mean = P.q_mean; qa.q_scale = P.q_scale; qa.q_codes = P.q_codes;
  qa.N = Dm.N; qa.Nk = Dm.Nk; qa.nQb = Dm.nQb; qa.block_groups = Dm.block_groups; qa.qg = Dm.qg;
  qa.qm = qm; qa.sm = sm; qa.q_corr = nullptr; qa.k_mean = P.k_mean; qa.G = Dm.H / Dm.Hkv; qa.kappa = Dm.kappa;
  qa.head_scale = nullptr; qa.stats_only = 0; qa.smooth_q = Dm.smooth_q; qa.k_sum = nullptr; qa.nchunk = (Dm.Nk + STAT_ROWS - 1) / STAT_ROWS; qa.smooth_k = Dm.smooth_k;
  qa.q_digits = Dm.ds_mode == DS_DIGITS && Dm.smooth_q ? P.q_digits : nullptr; qa.q_dscale = P.q_dscale;
  qa.narrow = qm.heads_inner && (long long)BH * Dm.nQb >= 512;
  QuantKV ka;
  ka.k = k; ka.v = v; ka.k_mean = P.k_mean; ka.v_scale = P.v_scale; ka.v_mean = v_mean;
  ka.k_scale = P.k_scale; ka.k_codes = P.k_codes; ka.v_codes = P.v_codes; ka.q_mean = P.q_mean; ka.delta_s = P.delta_s;
  ka.Nq = Dm.N; ka.Nk = Dm.Nk; ka.nKb = Dm.nKb; ka.nQb = Dm.nQb; ka.G = qa.G; ka.kappa = Dm.kappa;
  ka.block_groups = Dm.block_groups; ka.kg = Dm.kg; ka.causal = Dm.causal; ka.km = km; ka.sm = sm;
  ka.head_scale = nullptr; ka.stats_only = 0; ka.zero_ds = !Dm.smooth_q; ka.q_digits = P.q_digits; ka.q_dscale = P.q_dscale;
  ka.k_sum = P.k_sum; ka.v_max = P.v_max; ka.nchunk = (Dm.Nk + STAT_ROWS - 1) / STAT_ROWS; ka.smooth_k = Dm.smooth_k;
  ka.code_max = E4M3_MAX; ka.bounded = !Dm.stats_given; ka.parts = k_parts(Dm);
  // Taken one by one, K and V have every other XCD to themselves, on a grid that runs through the key blocks first.  That is the better
  // order (two kinds of code and of registers kept apart: 24 heads of 493 tokens, 8-bit, K and V 7.7 us mixed, 6.8 apart; 16 on 8 heads of
  // 1261 tokens of 256 channels, 4-bit, whole call 81.6, 80.2) unless K takes much longer than V and the chip is full.
  ka.mixed = INT4 && D < 256 && !km.heads_inner && (!few_rows(Dm) || (long long)BHkv * Dm.nKb >= 256);
  // K and V in one launch; `reduced`: mean(K) and delta_V are in place
  auto quant_kv = [&](bool reduced) {
    dim3 grid = block_grid(km, 2 * Dm.nKb, BHkv);
    grid.z = ka.parts;
#define SAGE_QKV(DSM_)                                                                                                  \
  do {                                                                                                                  \
    if (Dm.smooth_v) k_quant_kv<BF16, INT4, D, DSM_, true, false><<<grid, 256, 0, s>>>(ka);                              \
    else if (reduced) k_quant_kv<BF16, INT4, D, DSM_, false, false><<<grid, 256, 0, s>>>(ka);                            \
    else k_quant_kv<BF16, INT4, D, DSM_, false, true><<<grid, 256, 0, s>>>(ka);                                          \
  } while (0)
    if (INT4 && Dm.ds_mode == DS_FP64) SAGE_QKV(INT4 ? DS_FP64 : DS_DIGITS);
    else SAGE_QKV(DS_DIGITS);
#undef SAGE_QKV
  };
  if (small_call(Dm)) {
    // rows of 8 n workgroups all begin on the same XCD, of 8 n + 4 every other one, of an even number every fourth
    const int row = qa.G * Dm.nQb + (Dm.stats_given ? 0 : ka.nchunk), even = Dm.stats_given ? 1 : row & -row;
    const SmallStats st = {k, v, P.k_sum, P.v_max, ka.nchunk, km, even >= 8 ? 0 : (even == 4 ? 1 : 2), even >= 8 ? 7 : even - 1, 1.0f / (float)Dm.nQb};
    k_quant_q_and_stats<BF16, INT4, D><<<dim3(row, BHkv), 256, 0, s>>>(qa, st);
    quant_kv(Dm.stats_given);
    return hipGetLastError();
  }
  auto quant_q_pass = [&](float* corr, const float* head_scale, int stats_only, const Finalize* f = nullptr) {
    QuantQ x = qa;
    x.q_corr = corr; x.head_scale = head_scale; x.stats_only = stats_only;
    dim3 grid = block_grid(qm, Dm.nQb, BH);
    unsigned rows = 0;
    if (f) rows = ((f->n + FIN_ENT - 1) / FIN_ENT + grid.x - 1) / grid.x;
    grid.y += rows;
    k_quant_q<BF16, INT4, D><<<grid, 256, 0, s>>>(x, f ? *f : Finalize{}, rows);
  };
  auto quant_q = [&](const Finalize* f = nullptr) {
    float* corr = Dm.want_lse ? P.q_corr : nullptr;
    if (Dm.tensor_groups) {     // block scales, their maximum per head, then the codes with that one scale
      quant_q_pass(nullptr, nullptr, 1, f);
      k_head_scale<<<BH, 256, 0, s>>>(P.q_scale, P.q_head_scale, BQ / Dm.qg, Dm.nQb * (BQ / Dm.qg), BQ, Dm.H, 0, Dm.N,
                                     Dm.Nk, sm);
      quant_q_pass(corr, P.q_head_scale, 0);
    } else {
      quant_q_pass(corr, nullptr, 0, f);
    }
  };
  auto quant_k_pass = [&](const float* head_scale, int stats_only) {
    QuantKV x = ka;
    x.head_scale = head_scale; x.stats_only = stats_only;
    dim3 grid = block_grid(km, Dm.nKb, BHkv);
    grid.z = ka.parts;
#define SAGE_QK(DSM_) k_quant_k<BF16, INT4, D, DSM_><<<grid, 256, 0, s>>>(x)
    // (the 8-bit build has no Delta-S: one instantiation, named by the default mode)
    if (INT4 && Dm.ds_mode == DS_FP32) SAGE_QK(INT4 ? DS_FP32 : DS_DIGITS);
    else if (INT4 && Dm.ds_mode == DS_FP64) SAGE_QK(INT4 ? DS_FP64 : DS_DIGITS);
    else {
      SAGE_QK(DS_DIGITS);
    }
#undef SAGE_QK
  };
  // The partial statistics are finished under the quantization of Q (5 us as a launch of its own: 64 heads of 2048 tokens
  // 114.2 / 111.8 us, 64 on 8 of 3000 153.6 / 150.1, 32 of 8192, 8-bit mode 400 / 397).  With the log-sum-exp Q needs mean(K) itself and sums
  // the chunks in every workgroup: 4 chunks 39.4 / 37.2, 8 89.9 / 88.7, but 16 (512 queries) 84.7 / 85.5, 64 138 / 149.
  // Smooth V needs the sums before its second pass.  (With the statistics given, P.k_mean and P.v_scale are the caller's arrays.)
  const Finalize fin = finalize_args(Dm, P);
  const bool fin_with_q = !Dm.stats_given && !Dm.smooth_v && (!Dm.want_lse || fin.nchunk <= 8) && (long long)BH + fin.n / FIN_ENT + 2 <= 65535;
  if (fin_with_q && Dm.want_lse) qa.k_sum = P.k_sum;
  if (!Dm.stats_given && (fin_with_q || Dm.want_lse)) launch_stats_t<BF16, D>(Dm, P, s, !fin_with_q);
  quant_q(fin_with_q ? &fin : nullptr);
  if (!Dm.stats_given && !fin_with_q && !Dm.want_lse) launch_stats_t<BF16, D>(Dm, P, s);
  if (kv_pair(Dm)) {
    quant_kv(true);
    return hipGetLastError();
  }
  if (Dm.tensor_groups) {
    quant_k_pass(nullptr, 1);
    k_head_scale<<<BHkv, 256, 0, s>>>(P.k_scale, P.k_head_scale, BKV / Dm.kg, Dm.nKb * (BKV / Dm.kg), BKV, Dm.Hkv, 1,
                                     Dm.N, Dm.Nk, sm);
    quant_k_pass(P.k_head_scale, 0);
  } else {
    quant_k_pass(nullptr, 0);
  }
  const dim3 gv = block_grid(km, Dm.nKb, BHkv);
#define SAGE_QV(SV, PF) k_quant_v<BF16, D, SV, PF><<<gv, 256, 0, s>>>(ka)
  if (Dm.smooth_v) {
    if (Dm.pvf == PV_INT8) SAGE_QV(true, PV_INT8);
    else if (Dm.pvf == PV_E5M2) SAGE_QV(true, PV_E5M2);
    else SAGE_QV(true, PV_E4M3);
  } else {
    if (Dm.pvf == PV_INT8) SAGE_QV(false, PV_INT8);
    else if (Dm.pvf == PV_E5M2) SAGE_QV(false, PV_E5M2);
    else SAGE_QV(false, PV_E4M3);
  }
#undef SAGE_QV
  return hipGetLastError();
}

hipError_t launch_prologue(const Dims& D, const Ptrs& P, hipStream_t s) {
#define SAGE_PRO(BF, I4, DD) return launch_prologue_t<BF, I4, DD>(D, P, s)
  if (D.d == 256) {
    if (D.bf16) { if (D.int4) SAGE_PRO(true, true, 256); else SAGE_PRO(true, false, 256); }
    else        { if (D.int4) SAGE_PRO(false, true, 256); else SAGE_PRO(false, false, 256); }
  } else if (D.d == 128) {
    if (D.bf16) { if (D.int4) SAGE_PRO(true, true, 128); else SAGE_PRO(true, false, 128); }
    else        { if (D.int4) SAGE_PRO(false, true, 128); else SAGE_PRO(false, false, 128); }
  } else {
    if (D.bf16) { if (D.int4) SAGE_PRO(true, true, 64); else SAGE_PRO(true, false, 64); }
    else        { if (D.int4) SAGE_PRO(false, true, 64); else SAGE_PRO(false, false, 64); }
  }
#undef SAGE_PRO
}

hipError_t launch_kv_stats(const Dims& D, const Ptrs& P, hipStream_t s, bool finalize) {
  if (D.d == 256)      { if (D.bf16) launch_stats_t<true, 256>(D, P, s, finalize); else launch_stats_t<false, 256>(D, P, s, finalize); }
  else if (D.d == 128) { if (D.bf16) launch_stats_t<true, 128>(D, P, s, finalize); else launch_stats_t<false, 128>(D, P, s, finalize); }
  else                 { if (D.bf16) launch_stats_t<true, 64>(D, P, s, finalize); else launch_stats_t<false, 64>(D, P, s, finalize); }
  return hipGetLastError();
}

template <bool BF16, int D>
static void launch_stats_update_t(const Dims& Dm, const Ptrs& P, double* state_sum, float* state_max, int fresh,
                                  long long n_total, hipStream_t s) {
  const int BHkv = Dm.B * Dm.Hkv, nstat = BHkv * Dm.d;
  const TensorMap km = make_tensor_map(Dm.nhd, Dm.Hkv, Dm.Nk, Dm.d, false);
  const int nchunk = (Dm.Nk + STAT_ROWS - 1) / STAT_ROWS;
  const dim3 gstat = block_grid(km, nchunk, BHkv);
  const float code_max = Dm.pvf == PV_INT8 ? INT8_PV_MAX : (Dm.pvf == PV_E5M2 ? E5M2_MAX : E4M3_MAX);
  k_col_stats<BF16, D, false><<<gstat, 256, 0, s>>>((const unsigned short*)P.k, (const unsigned short*)P.v, P.k_sum, nullptr,
                                                    P.v_max, Dm.N, Dm.Nk, km, Dm.seq);
  k_accumulate_stats<<<(nstat + FIN_ENT - 1) / FIN_ENT, FIN_ENT * FIN_PARTS, 0, s>>>(P.k_sum, P.v_max, state_sum, state_max, P.k_mean, P.v_scale, nstat,
                                                         Dm.d, nchunk, fresh, n_total, code_max);
}

hipError_t launch_kv_stats_update(const Dims& D, const Ptrs& P, double* state_sum, float* state_max, int fresh,
                                  long long n_total, hipStream_t s) {
#define SAGE_SU(BF, DD) launch_stats_update_t<BF, DD>(D, P, state_sum, state_max, fresh, n_total, s)
  if (D.d == 256)      { if (D.bf16) SAGE_SU(true, 256); else SAGE_SU(false, 256); }
  else if (D.d == 128) { if (D.bf16) SAGE_SU(true, 128); else SAGE_SU(false, 128); }
  else                 { if (D.bf16) SAGE_SU(true, 64); else SAGE_SU(false, 64); }
#undef SAGE_SU
  return hipGetLastError();
}

hipError_t launch_unpack(const Dims& D, const Ptrs& P, const void* quant_out, hipStream_t s) {
  const sage_quant_out& qo = *(const sage_quant_out*)quant_out;
  struct { int8_t *qc, *kc; uint8_t* vc; float *qs, *ks, *vs, *km, *qm, *ds, *vm; } o = {
      qo.q_codes, qo.k_codes, qo.v_codes, qo.q_scale, qo.k_scale, qo.v_scale, qo.k_mean, qo.q_mean, qo.delta_s,
      qo.v_mean};
  const int BH = D.B * D.H, BHkv = D.B * D.Hkv;
  const unsigned gx = (unsigned)(((size_t)D.N * D.d + 255) / 256), gxk = (unsigned)(((size_t)D.Nk * D.d + 255) / 256);
  if (o.qc) k_unpack_codes<<<dim3(gx, BH), 256, 0, s>>>(P.q_codes, o.qc, D.N, D.d, D.nQb * q_slab_bytes(D.d, D.int4), 0, D.int4);
  if (o.kc) k_unpack_codes<<<dim3(gxk, BHkv), 256, 0, s>>>(P.k_codes, o.kc, D.Nk, D.d, D.nKb * k_block_bytes(D.d, D.int4), 1, D.int4);
  if (o.vc) k_unpack_codes<<<dim3(gxk, BHkv), 256, 0, s>>>((const int8_t*)P.v_codes, (int8_t*)o.vc, D.Nk, D.d, (size_t)D.nKb * BKV * D.d, 2, 0);
  const int nqg = (D.N + D.qg - 1) / D.qg, nkg = (D.Nk + D.kg - 1) / D.kg;
  if (o.qs) k_unpack_rows<<<dim3((nqg + 255) / 256, BH), 256, 0, s>>>(P.q_scale, o.qs, nqg, D.nQb * (BQ / D.qg));
  if (o.ks) k_unpack_rows<<<dim3((nkg + 255) / 256, BHkv), 256, 0, s>>>(P.k_scale, o.ks, nkg, D.nKb * (BKV / D.kg));
  if (o.vs) k_unpack_rows<<<dim3(1, BHkv), 256, 0, s>>>(P.v_scale, o.vs, D.d, D.d);
  if (o.km) k_unpack_rows<<<dim3(1, BHkv), 256, 0, s>>>(P.k_mean, o.km, D.d, D.d);
  if (o.vm && D.smooth_v) k_unpack_rows<<<dim3(1, BHkv), 256, 0, s>>>(P.v_mean, o.vm, D.d, D.d);
  if (D.int4) {
    if (o.qm) k_unpack_rows<<<dim3(1, BH * D.nQb), 256, 0, s>>>(P.q_mean, o.qm, D.d, D.d);
    if (o.ds) k_unpack_rows<<<dim3((D.Nk + 255) / 256, BH * D.nQb), 256, 0, s>>>(P.delta_s, o.ds, D.Nk, D.nKb * BKV);
  }
  return hipGetLastError();
}

}  // namespace sage
