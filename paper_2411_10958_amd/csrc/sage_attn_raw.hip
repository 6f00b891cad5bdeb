// Attention straight from K and V, for calls in which every key block meets one tile of at most 32 query columns: decode
// steps and very short query chunks.  There the general path reads K and V, writes their codes, reads the codes and the
// Delta-S rows again and spends most of its time on that traffic; here a workgroup quantizes a 64-key block on its way
// into LDS and uses it there, so K and V are read once after the statistics pass (or once in all, with the statistics
// supplied) and nothing of their size is written.  The few query rows are quantized by the workgroups themselves too.
// Same groups, scales, codes, Delta-S and chunk rule as the general path, and the same order of every float64 sum: which of the
// two serves a call depends on how many workgroups it makes, its results must not.
#include "sage_attn_core.h"
#include "sage_quant.h"

#include <type_traits>

namespace sage {

struct RawParams {
  const unsigned short *q, *k, *v;   // (q is laid out like the output)
  const float* k_mean;               // mean(K) per KV head
  float* q_corr;                     // where the row constants of the log-sum-exp go for the merge
  const double* k_sum;               // not null: mean(K) and delta_V are not there yet, these are the partial results of the statistics
  const unsigned* v_max;             // pass; the workgroup reduces its head's, and a head's first one writes delta_V for the merge
  float* v_scale;
  int nchunk;
  TensorMap km;
};

// x[0] + ... + x[N - 1], neighbours first.
template <int N>
__device__ __forceinline__ double pair_sum(double (&x)[N]) {
#pragma unroll
  for (int m = 1; m < N; m *= 2) {
#pragma unroll
    for (int i = 0; i + m < N; i += 2 * m) x[i] += x[i + m];
  }
  return x[0];
}

// One workgroup (8 wavefronts): one chunk of the key blocks of one (batch, KV head).  Column c of the tile is query c % n of
// head c / n of the KV head's group (n: the sequence's query count).
//
// Wavefronts 0..3 quantize K, 4 and 5 V: a block's raw rows are in registers (requested a block ahead, as soon as the previous
// ones are unpacked), are smoothed, quantized and written to LDS in the order the matrix operands are read in.  Wavefronts 6 and
// 7 attend: each forms the block's scores and P~ for all 32 columns - the same values in both - and multiplies them
// with its own half of the channels of V^.  LDS holds two blocks, one barrier per block.
//
// Bound: each block is a chain of its wavefronts' work behind one barrier; the split above is what makes the longest of them short,
// and keeps every part in 128 registers (d = 64 and 128; d = 256: 189), so that two workgroups share a CU. 4 x 8 KV heads, 32768 keys,
// d = 128, one query, statistics supplied, the kernel alone: 81 us in the 4-bit mode (LONE; 537 MB: 6.6 TB/s), 83 in the 8-bit one (6.5 TB/s),
// and a merge of 5 us; whole calls 94 and 98, with two queries 116 and 98.  Whole calls of earlier forms, both modes: quantizers and attention kernel 255 / 185, four wavefronts quantizing both and four attending, with
// 16 spilled registers, rows addressed and padded lane by lane and every mean of Delta-S waited for by itself 153 / 122, those mended
// 139 / 103 with two attending wavefronts instead of four, this form 101 / 88. 16 of 256 channels, 30000 keys, 4-bit: 147, 128, 114.
// 16 x 16 of 64 channels, 5003 keys, 8-bit: 139, 82, 74.  Tried: one attending wavefront (d = 64: 71 -> 69 us on grouped heads, 74 ->
// 77 on ungrouped ones); four for V at d = 256 (128 -> 128, 8-bit 70 -> 82).  K by 64-byte pieces of four lanes and an exchange in
// registers pays at d = 256 only, where a lane's own piece is a whole cache line (quad_exchange).
// HEADS: 4, or PACK_G where the 4-bit mode has more than four query heads per KV head (two chains of the Delta-S product).
// LONE: one query per head in the 4-bit mode.  It is its own block mean, gamma(Q) = 0, so all of its codes are 0 and so is
// their product with K's: the score is Delta-S, and neither codes nor scales of Q and K are formed.  Same bits; whole calls, the kernel with
// the codes / this one, on inputs in turn: 4 x 8 KV heads of 32768 keys 194 / 182 us, statistics supplied 115 / 94, 16 x 16
// of 64 channels, 5003 keys 95 / 74, 16 of 256, 30000 keys 119 / 100, 8 of 4000 keys, statistics not supplied, 34 / 30.  (A branch in the one kernel spilled 38 registers
// of the calls with more queries: 70 / 87.)
constexpr int RAW_V = 2, RAW_ATT = 2, RAW_THREADS = 64 * (4 + RAW_V + RAW_ATT);
template <int D, bool INT4, bool CAUSAL, bool BF16, int HEADS, bool LONE = false>
__global__ void __launch_bounds__(RAW_THREADS, D == 256 ? 2 : 4) k_attn_raw(const AttnParams p, const RawParams x) {
  static_assert(!LONE || (INT4 && !CAUSAL), "one query sees every key");
  constexpr int CPL = D / 4;                                     // K: channels per lane
  constexpr int NCG = D / 8, NRG = 64 * RAW_V / NCG, RPT = BKV / NRG;   // V: 8 channels of RPT keys per thread
  constexpr int CT = D / 32, CTW = CT / RAW_ATT;                 // channel tiles of the output, per attending wavefront
  constexpr int KCK = (int)(k_block_bytes(D, INT4) / 16), KC = D * BKV / 16;
  constexpr int QMAX = INT4 ? 7 : 127;
  constexpr int NP = qk_pieces<D, INT4>();
  constexpr int QMS = CPL + 2;     // doubles per (head, channel quarter) in s_qm: 16 of them start in 16 different bank groups
  __shared__ v4i s_k[2][KCK];
  __shared__ v4i s_v[2][KC];
  __shared__ __align__(16) float s_ds[INT4 ? 2 : 1][INT4 ? HEADS : 1][BKV];
  __shared__ __align__(16) double s_qm[INT4 ? HEADS * 4 * QMS : 2];
  __shared__ __align__(16) float s_km[D], s_vs[D], s_vi[D];      // mean(K); delta_V and its reciprocal (0: divide)
  __shared__ float s_ks[2][4];

  const int t = threadIdx.x, lane = t & 63;
  const int wave = __builtin_amdgcn_readfirstlane(t >> 6);
  const bool k_wave = wave < 4, v_wave = !k_wave && wave < 4 + RAW_V;
  const int w = k_wave ? wave : wave - 4 - RAW_V;                // (of the K quantizers, or of the attending wavefronts)
  const int n = lane & 31, half = lane >> 5;
  const int split = blockIdx.x % p.splits, tile = blockIdx.x / p.splits;
  const int G = p.H / p.Hkv;
  const int b = tile / p.Hkv, h = (tile - b * p.Hkv) * G;        // the group's first query head
  const size_t bh = (size_t)b * p.H + h, bhkv = tile;
  const Seq sq = seq_of(p.seq, (unsigned)b, p.N, p.Nk);
  if (sq.n <= 0) return;
  const int col = n, cols = G * sq.n;                            // (cols <= 32: the launch rule)
  const bool col_ok = col < cols;
  const int hq = col_ok ? col / sq.n : 0, query = col_ok ? col - hq * sq.n : 0;
  if (sq.nk == 0) {                                              // no keys at all: the rows are defined as zeros
    if (split != 0) return;
    for (int idx = t; idx < cols * (D / 8); idx += RAW_THREADS) {
      const int c = idx / (D / 8), g = c / sq.n, r = c - g * sq.n;
      unsigned short* o = reinterpret_cast<unsigned short*>(p.out) + row_offset(p.om, head_offset(p.om, (unsigned)(bh + g)), (int)sq.q0 + r);
      *reinterpret_cast<uint4*>(o + (idx % (D / 8)) * 8) = make_uint4(0u, 0u, 0u, 0u);
    }
    if (p.lse && t < cols) p.lse[lse_index(p, sq, b, h + t / sq.n, t % sq.n)] = -INFINITY;
    return;
  }
  int j0, j1;
  {
    int nblk = (sq.nk + BKV - 1) / BKV;
    if (CAUSAL) nblk = min(nblk, (BQ - 1 + sq.coff) / BKV + 1);
    const int n_vis = CAUSAL ? min(nblk, sq.coff / BKV + 1) : nblk;
    const KeyChunk kc = key_chunk(split, p.splits, nblk, n_vis);
    j0 = kc.j0;
    j1 = kc.j1;
  }
  if (j0 >= j1) {                                                // an empty chunk: offset -inf, sum 0 (the merge skips it)
    if (t < BQ) {
      float* el = p.part_el + ((size_t)blockIdx.x * BQ + t) * 2;
      el[0] = -INFINITY; el[1] = 0.0f;
    }
    return;
  }

  if (x.k_sum) {
    // finalize_stats_block for one head: RAW_THREADS / D threads to a channel (the sums are exact, whatever their order)
    constexpr int PARTS = RAW_THREADS / D;
    static_assert(PARTS * D == RAW_THREADS && sizeof(s_v) >= RAW_THREADS * 12, "the parts meet where V's codes will be");
    double* sum = reinterpret_cast<double*>(&s_v[0][0]);
    float* max = reinterpret_cast<float*>(sum + RAW_THREADS);
    const int c = t % D, part = t / D;
    const size_t p0 = (size_t)bhkv * x.nchunk * D + c;
    double ks = 0.0;
    float vm = 0.0f;
#pragma unroll 4
    for (int ch = part; ch < x.nchunk; ch += PARTS) {
      ks += x.k_sum[p0 + (size_t)ch * D];
      vm = fmaxf(vm, __uint_as_float(x.v_max[p0 + (size_t)ch * D]));
    }
    sum[t] = ks; max[t] = vm;
    __syncthreads();
    if (t < D) {
#pragma unroll
      for (int i = 1; i < PARTS; ++i) { ks += sum[i * D + t]; vm = fmaxf(vm, max[i * D + t]); }
      s_km[t] = (float)(ks / (double)sq.nk);
      const float vs = __fdiv_rn(vm, E4M3_MAX);
      s_vs[t] = vs;
      s_vi[t] = div_by_ok(vs) ? __fdiv_rn(1.0f, vs) : 0.0f;
      if (split == 0) x.v_scale[bhkv * D + t] = vs;
    }
  } else {
    for (int c = t; c < D; c += RAW_THREADS) {
      s_km[c] = x.k_mean[bhkv * D + c];
      const float vs = p.v_scale[bhkv * D + c];
      s_vs[c] = vs;
      s_vi[c] = div_by_ok(vs) ? __fdiv_rn(1.0f, vs) : 0.0f;
    }
  }
  if constexpr (INT4) {
    for (int idx = t; idx < HEADS * D; idx += RAW_THREADS) {
      const int g = idx / D, c = idx % D;
      // block mean of the head's queries (one block: at most 32), added in quant_q4_block's order
      double mean = 0.0;
      if (g < G) {
        constexpr int RG = D / 16, NG = 32 / RG;             // rows are summed in runs of RG, the runs in pairs
        const unsigned short* qh = x.q + row_offset(p.om, head_offset(p.om, (unsigned)(bh + g)), (int)sq.q0) + c;
        double run[NG];
#pragma unroll
        for (int k = 0; k < NG; ++k) {
          run[k] = 0.0;
          for (int r = RG * k; r < min(sq.n, RG * (k + 1)); ++r) run[k] += (double)load16<BF16>(qh[(size_t)r * (size_t)p.om.sn]);
        }
        mean = (double)(float)(pair_sum(run) / (double)sq.n);
      }
      s_qm[(g * 4 + c / CPL) * QMS + c % CPL] = mean;
    }
  }
  __syncthreads();

  const size_t hbase = head_offset(x.km, (unsigned)bhkv) + sq.k0 * (size_t)x.km.sn;
  // Rows of block j: a uniform base and 32-bit lane offsets, formed once (64 rows of a token-major tensor stay below 2^32
  // bytes).  Where the sequence ends inside the block its last row stands in for the rows behind it; their
  // codes are cleared below (K) or meet a P~ of zero (V).  Past the chunk its last block is read once more, and not used.
  const unsigned rowb = 2u * (unsigned)x.km.sn;
  // K as in k_quant_k: lane l of wavefront w holds key 16 w + l % 16, channels CPL (l / 16) ..
  const int kk = lane >> 4, c0 = CPL * kk, kr = 16 * w + (lane & 15);
  const unsigned koff = (unsigned)kr * rowb + (D == 256 ? 16 * kk : 2 * c0);
  constexpr int KSTEP = D == 256 ? 64 : 16;                // bytes from one of the lane's loads to the next (256: quad_piece)
  uint4 rk[CPL / 8];
  auto fetch_k = [&](int j) {
    j = min(j, j1 - 1);
    const char* base = reinterpret_cast<const char*>(x.k + row_offset(x.km, hbase, j * BKV));
    const int last = sq.nk - 1 - j * BKV;
    unsigned off = koff;
    if (last < BKV - 1) off -= (unsigned)max(kr - last, 0) * rowb;
#pragma unroll
    for (int i = 0; i < CPL / 8; ++i) rk[i] = *reinterpret_cast<const uint4*>(base + KSTEP * i + off);
  };
  auto quant_k = [&](int j, int cur) {
    // smooth, group maximum over the wavefront's 16 keys, codes and scale (k_quant_k's arithmetic)
    float xk[CPL];
    float mx = 0.0f;
    if constexpr (D == 256) quad_exchange(rk);
#pragma unroll
    for (int i = 0; i < CPL / 8; ++i) {
      unpack8<BF16>(rk[i], &xk[8 * i]);
      const float4 m0 = *reinterpret_cast<const float4*>(&s_km[c0 + 8 * i]);
      const float4 m1 = *reinterpret_cast<const float4*>(&s_km[c0 + 8 * i + 4]);
      const float mean[8] = {m0.x, m0.y, m0.z, m0.w, m1.x, m1.y, m1.z, m1.w};
#pragma unroll
      for (int e = 0; e < 8; ++e) xk[8 * i + e] = __fsub_rn(xk[8 * i + e], mean[e]);
    }
    __builtin_amdgcn_sched_barrier(0);
    fetch_k(j + 1);                    // (the registers are free; in flight under the rest of this block's work)
    if (j * BKV + BKV > sq.nk && j * BKV + kr >= sq.nk) {        // padded keys: codes 0, Delta-S 0
#pragma unroll
      for (int e = 0; e < CPL; ++e) xk[e] = 0.0f;
    }
    float delta = 0.0f;
    CodeScale qs;
    if constexpr (!LONE) {
#pragma unroll
      for (int e = 0; e < CPL; ++e) mx = fmaxf(mx, fabsf(xk[e]));
      delta = __fdiv_rn(wave_max(mx), (float)QMAX);
      if (lane == 0) s_ks[cur][w] = delta;
      qs = code_scale(delta);
    }
    uint8_t* img = reinterpret_cast<uint8_t*>(&s_k[cur][0]);
    if constexpr (INT4) {
      // Delta-S: q_bar_g . gamma(K)_t in float64, four heads at a time by v_mfma_f64_4x4x4_4b_f64: four independent
      // 4 x 4 products per instruction, lane l supplies A[l % 4][l / 16] and B[l / 16][l % 4] of product (l / 4) % 4 and
      // receives D[l / 16][l % 4].  Product i holds keys 16 w + 4 i + 0..3, contraction slot (step cs, l / 16) channel
      // CPL (l / 16) + cs: the lane's own registers, in order.  (The 16-row form of the
      // general path spends 2048 matrix cycles per block on rows that a few heads leave empty; this one 512 per 4 heads.)
      // One chain of accumulations, in the general path's order: with two, which are a little shorter, a Delta-S that
      // lies next to the middle of two FP32 values could round to the other one (decode of 32768 keys: 249 us either way).
      const double kap = (double)p.kappa;
      const double* qa = &s_qm[((lane & 3) * 4 + kk) * QMS];
      // The means come out of LDS a chunk of channels ahead of their use: read one by one, each product waited for its own
      // (32768 keys, 4-bit mode 145 us, 139); the two chains of five to eight heads run side by side.
      constexpr int NCH = HEADS / 4, CH = (D == 256 ? 4 : 8) / NCH;
      double acc[NCH], qv[2][NCH][CH];
      auto means = [&](int c, int b) {
#pragma unroll
        for (int i = 0; i < NCH; ++i) {
#pragma unroll
          for (int e = 0; e < CH; ++e) qv[b][i][e] = qa[16 * i * QMS + c + e];
        }
      };
#pragma unroll
      for (int i = 0; i < NCH; ++i) acc[i] = 0.0;
      means(0, 0);
#pragma unroll
      for (int cs = 0; cs < CPL; cs += CH) {
        if (cs + CH < CPL) means(cs + CH, (cs / CH + 1) & 1);
        asm volatile("" ::: "memory");                 // (not all of them at once)
#pragma unroll
        for (int e = 0; e < CH; ++e) {
          asm volatile("" : "+v"(xk[cs + e]));         // (widened as it is used)
          const double xd = (double)xk[cs + e];
#pragma unroll
          for (int i = 0; i < NCH; ++i) acc[i] = __builtin_amdgcn_mfma_f64_4x4x4f64(qv[(cs / CH) & 1][i][e], xd, acc[i], 0, 0, 0);
        }
      }
#pragma unroll
      for (int i = 0; i < NCH; ++i) {
        double s = kap * acc[i];
        // (an infinite key, which supplied statistics allow, makes its group's scale infinite and 0 codes times that NaN: so must the
        // score be that leaves both out)
        if constexpr (LONE) s = __builtin_fma(0.0, acc[i], s);
        s_ds[cur][4 * i + kk][kr] = (float)s;
      }
      if constexpr (LONE) return;
      constexpr int NPL = CPL > 32 ? CPL / 32 : 1, CPP = CPL / NPL;
#pragma unroll
      for (int pl = 0; pl < NPL; ++pl) {
        Codes32 cd;
        if constexpr (CPP < 32) {
#pragma unroll
          for (int e = 0; e < 16; ++e) { cd.ev[e] = 0.0f; cd.od[e] = 0.0f; }
        }
        code_group<CPP, QMAX>(xk + CPP * pl, delta, qs, [&](int e, float c) { cd.set(e, c); });
        const v6u pw = cd.pack();
        int lane_m, e0;
        const size_t op = k_op6(kr, c0 + CPP * pl, D, &lane_m, &e0);
        const int d0 = (6 * e0) >> 5;
#pragma unroll
        for (int i = 0; i < CPP * 6 / 32; ++i)
          *reinterpret_cast<unsigned*>(img + op + op6_byte(lane_m, 4 * (d0 + i))) = pw[i];
      }
    } else {
#pragma unroll
      for (int i = 0; i < CPL / 16; ++i) {
        unsigned c[16];
        code_group_bytes<16, QMAX>(xk + 16 * i, delta, qs, c);
        *reinterpret_cast<uint4*>(img + k_code_off(kr, c0 + 16 * i, D)) = pack16(c);
      }
    }
  };
  // V: codes of four consecutive keys of a channel side by side, NH such runs per thread
  constexpr int HR = 4, NH = RPT / HR;
  const int tv = t - 256, cg = tv % NCG, vr = HR * (tv / NCG);
  const unsigned voff = (unsigned)vr * rowb + 16 * cg;
  uint4 rv[NH][HR];
  bool v_fast = true;
  auto fetch_v = [&](int j, uint4 (&rows)[HR], int hh) {
    j = min(j, j1 - 1);
    const char* base = reinterpret_cast<const char*>(x.v + row_offset(x.km, hbase, j * BKV));
    const int last = sq.nk - 1 - j * BKV, r0 = HR * NRG * hh;
    unsigned off[HR], vo = voff;
    asm volatile("" : "+v"(vo));         // (added up for every block: kept, the offsets cost a register each)
#pragma unroll
    for (int i = 0; i < HR; ++i) off[i] = vo + (unsigned)(r0 + i) * rowb;
    if (last < BKV - 1) {
#pragma unroll
      for (int i = 0; i < HR; ++i) off[i] -= (unsigned)max(vr + r0 + i - last, 0) * rowb;
    }
#pragma unroll
    for (int i = 0; i < HR; ++i) rows[i] = nt_load16(reinterpret_cast<const unsigned short*>(base + off[i]));
  };
  // Channel c's 16-byte chunks are XOR-ed in their place by (c / 16) % 8, so that the 16 channel groups of a store meet 16
  // different bank groups; the thread's eight channels are eight neighbouring chunks, XOR-ed alike
  static_assert(NH == 1 || HR * NRG == 32 || HR * NRG == 16, "a further run of keys is 16 or 32 keys on: 32 or 64 chunks");
  const unsigned vdst = (unsigned)v_code_off(vr, 8 * cg, D) ^ (unsigned)(((cg >> 1) & 7) * 16);
  auto quant_v = [&](int j, int cur) {
    uint8_t* img = reinterpret_cast<uint8_t*>(&s_v[cur][0]);
    unsigned vd = vdst;
    asm volatile("" : "+v"(vd));
    float vs[8], vi[8];
#pragma unroll
    for (int e = 0; e < 8; ++e) { vs[e] = s_vs[8 * cg + e]; vi[e] = s_vi[8 * cg + e]; }
#pragma unroll
    for (int hh = 0; hh < NH; ++hh) {
      float xv[HR][8];
#pragma unroll
      for (int i = 0; i < HR; ++i) unpack8<BF16>(rv[hh][i], xv[i]);
      // (unpacked here and not in the two branches below: the rows' registers would not be free for the next block's, and a
      // copy at the end of the block would wait for those)
#pragma unroll
      for (int i = 0; i < HR; ++i) {
#pragma unroll
        for (int e = 0; e < 8; ++e) asm volatile("" : "+v"(xv[i][e]));
      }
      __builtin_amdgcn_sched_barrier(0);
      fetch_v(j + 1, rv[hh], hh);
      if (v_fast) {
#pragma unroll
        for (int i = 0; i < HR; ++i) {
#pragma unroll
          for (int e = 0; e < 8; ++e) xv[i][e] = div_by(xv[i][e], vs[e], vi[e]);
        }
      } else {
#pragma unroll
        for (int i = 0; i < HR; ++i) {
#pragma unroll
          for (int e = 0; e < 8; ++e) {
            xv[i][e] = vs[e] > 0.0f ? __fdiv_rn(xv[i][e], vs[e]) : 0.0f;
            asm volatile("" : "+v"(xv[i][e]) :: "memory");     // (one division at a time)
          }
        }
      }
#pragma unroll
      for (int e = 0; e < 8; ++e) {
        const unsigned off = (vd ^ (16u * e)) + 32u * HR * NRG * hh;
        // (the first conversion of the word keeps the other half of any register: one that is free afterwards)
        int wd = __builtin_amdgcn_cvt_pk_fp8_f32(xv[0][e], xv[1][e], __float_as_int(xv[0][e]), false);
        wd = __builtin_amdgcn_cvt_pk_fp8_f32(xv[2][e], xv[3][e], wd, true);
        *reinterpret_cast<int*>(img + off) = wd;
      }
      __builtin_amdgcn_sched_barrier(0);
    }
  };
  // (one barrier per block: block j is in LDS, and the other wavefronts are done with block j - 1)
  if (k_wave) {
    fetch_k(j0);
    for (int j = j0, cur = 0; j < j1; ++j, cur ^= 1) { quant_k(j, cur); __syncthreads(); }
    return;
  }
  if (v_wave) {
#pragma unroll
    for (int hh = 0; hh < NH; ++hh) fetch_v(j0, rv[hh], hh);
#pragma unroll
    for (int e = 0; e < 8; ++e) v_fast = v_fast && (s_vi[8 * cg + e] != 0.0f || s_vs[8 * cg + e] == 0.0f);   // (an all-zero channel: 0 * 0 = 0 either way)
    for (int j = j0, cur = 0; j < j1; ++j, cur ^= 1) { quant_v(j, cur); __syncthreads(); }
    return;
  }

  // ---- the wavefront's Q^ operands: both hold the same 32 columns and quantize them themselves (a separate launch for so
  // few rows costs 7 us: 16 x 8 KV heads, 5003 keys, 8-bit mode 85 / 79 us, 4 x 8, 32768 keys, 4-bit 263 / 243; 16 of 256 channels,
  // 30000 keys, 4-bit 238 / 231).  Lane (n, half)
  // supplies, of its column's query, PC consecutive channels per operand: smoothed
  // (4-bit mode), scale from the pair of queries, codes as quant_q4_block / quant_q8_block give them.
  constexpr int PC = INT4 ? 32 : 16;
  typename QkOperand<INT4>::type qreg[NP];
  float dq = 0.0f;
#pragma unroll
  for (int s = 0; s < NP; ++s) qreg[s] = typename QkOperand<INT4>::type{};
  if constexpr (!LONE) {
    const unsigned short* qrow = x.q + row_offset(p.om, head_offset(p.om, (unsigned)(bh + hq)), (int)sq.q0 + query);
    float mx = 0.0f;
    // one operand's channels at a time, fetched once for the maximum and again for the codes: kept, the row would cost a
    // wide head its registers for the whole kernel
    auto fetch = [&](int s, float (&xq)[PC]) {
      const int cq = (2 * s + half) * PC;
#pragma unroll
      for (int i = 0; i < PC / 8; ++i) unpack8<BF16>(*reinterpret_cast<const uint4*>(qrow + cq + 8 * i), &xq[8 * i]);
    };
    auto smooth = [&](int s, float (&xq)[PC]) {
      const int cq = (2 * s + half) * PC;
      if constexpr (INT4) {
#pragma unroll
        for (int e = 0; e < PC; ++e) {
          xq[e] = __fsub_rn(xq[e], (float)s_qm[(hq * 4 + (cq + e) / CPL) * QMS + (cq + e) % CPL]);
          if (e % 8 == 7) asm volatile("" ::: "memory");     // (not all of the means out of LDS at once)
        }
      }
    };
#pragma unroll
    for (int s = 0; s < NP; ++s) {
      float xq[PC];
      fetch(s, xq);
      smooth(s, xq);
#pragma unroll
      for (int e = 0; e < PC; ++e) mx = fmaxf(mx, fabsf(xq[e]));
      asm volatile("" ::: "memory");
    }
    mx = butterfly_max<32>(mx);
    const int other = (query ^ 1) < sq.n ? hq * sq.n + (query ^ 1) : hq * sq.n + query;      // column of the pair's other query
    dq = __fdiv_rn(fmaxf(mx, __shfl(mx, other, 64)), (float)QMAX);
    const bool fast = __builtin_amdgcn_ballot_w64(!(div_by_ok(dq) || dq == 0.0f)) == 0;      // (scale 0: all values are 0)
    const float rq = fast && dq > 0.0f ? __fdiv_rn(1.0f, dq) : 0.0f;
    auto codes = [&](float (&v)[PC]) {                     // v: values, then their codes
      if (fast) {
#pragma unroll
        for (int e = 0; e < PC; ++e) v[e] = rintf(div_by(v[e], dq, rq));
      } else {
#pragma unroll
        for (int e = 0; e < PC; ++e) {
          v[e] = (float)quant_code(v[e], dq, QMAX);
          asm volatile("" : "+v"(v[e]) :: "memory");       // (one division at a time)
        }
      }
    };
#pragma unroll
    for (int s = 0; s < NP; ++s) {
      float xq[PC];
      fetch(s, xq);
      smooth(s, xq);
      codes(xq);
      if constexpr (INT4) {
        Codes32 cd;
#pragma unroll
        for (int e = 0; e < PC; ++e) cd.set(e, xq[e]);
        const v6u pw = cd.pack();
#pragma unroll
        for (int i = 0; i < 8; ++i) qreg[s][i] = i < 6 ? (int)pw[i < 6 ? i : 0] : 0;
      } else {
#pragma unroll
        for (int i = 0; i < 4; ++i) {
          unsigned wd = 0;
#pragma unroll
          for (int e = 0; e < 4; ++e) wd |= ((unsigned)(int)xq[4 * i + e] & 0xffu) << (8 * e);
          qreg[s][i] = (int)wd;
        }
      }
      asm volatile("" ::: "memory");
    }
  }
  constexpr int DW = 32 * CTW;                                   // this wavefront's channels: DW w ..
  RowState<DW> st;
#pragma unroll
  for (int ct = 0; ct < CTW; ++ct) {
#pragma unroll
    for (int v = 0; v < 16; ++v) st.O[ct][v] = 0.0f;
  }
  st.m_run = -INFINITY;
  st.l_run = 0.0f;
  float m_sub = -INFINITY;
  int n_plain = min(j1, sq.nk / BKV);                            // blocks that need no mask
  if (CAUSAL) n_plain = min(n_plain, (sq.coff + 1) / BKV);
  const int n_keys_end = min(sq.nk, j1 * BKV);
  for (int j = j0, cur = 0; j < j1; ++j, cur ^= 1) {
    __syncthreads();
    v8i pb;
    float alpha;
    auto attend = [&](auto masked_) {
      constexpr bool MASKED = decltype(masked_)::value;
      Factors<0> fac;
      fac.c[0] = fac.c[1] = 0.0f;
      const int key0 = j * BKV, last = query + sq.coff;
      v16i raw[2], sc[2];
      auto lone_tile = [&](auto kt_) {
        constexpr int KT = decltype(kt_)::value;
        const float* dsr = &s_ds[cur][hq][32 * KT + 16 * half];
#pragma unroll
        for (int v = 0; v < 16; ++v) {
          float s = dsr[v];
          const int key = key0 + 32 * KT + 16 * half + v;
          if (MASKED && (key >= n_keys_end || (CAUSAL && key > last))) s = -INFINITY;
          sc[KT][v] = __float_as_int(s);
        }
      };
      // one key tile after the other, so that one tile's operands and raw scores are live at a time
      auto key_tile = [&](auto kt_) {
        constexpr int KT = decltype(kt_)::value;
        typename KBlockRegs<D, INT4>::type ka;
#pragma unroll
        for (int sp = 0; sp < NP; ++sp) ka[2 * sp + KT] = load_qk_operand<INT4>(&s_k[cur][0], 2 * sp + KT, lane);
        qk_key_tile<D, INT4, KT>(ka, qreg, raw);
        asm volatile("" ::: "memory");     // Delta-S is read after the operands of the product, into registers they leave
        if constexpr (INT4) {
          const v4f* dsv = reinterpret_cast<const v4f*>(&s_ds[cur][hq][32 * KT + 16 * half]);
#pragma unroll
          for (int g = 0; g < 4; ++g) {
            const v4f t4 = dsv[g];
#pragma unroll
            for (int r = 0; r < 4; ++r) sc[KT][4 * g + r] = __float_as_int(t4[r]);
          }
        }
        dequant_group<INT4, CAUSAL, MASKED, 0, KT, 0>(raw, sc, fac, half, key0, last, n_keys_end);
        dequant_group<INT4, CAUSAL, MASKED, 0, KT, 1>(raw, sc, fac, half, key0, last, n_keys_end);
        dequant_group<INT4, CAUSAL, MASKED, 0, KT, 2>(raw, sc, fac, half, key0, last, n_keys_end);
        dequant_group<INT4, CAUSAL, MASKED, 0, KT, 3>(raw, sc, fac, half, key0, last, n_keys_end);
        __builtin_amdgcn_sched_barrier(0);
      };
      if constexpr (LONE) {
        lone_tile(std::integral_constant<int, 0>{});
        lone_tile(std::integral_constant<int, 1>{});
      } else {
        KeyScales<0> ks;
        ks.s[0] = s_ks[cur][half];
        ks.s[1] = s_ks[cur][2 + half];
        fac.set(dq, p.kappa, ks);
        key_tile(std::integral_constant<int, 0>{});
        key_tile(std::integral_constant<int, 1>{});
      }
      alpha = update_max<DW, INT4, 0, PV_E4M3>(st, sc, fac, m_sub);
      float ls = 0.0f;
      exp_group<INT4, MASKED, 0, PV_E4M3, 0, 0>(sc, fac, m_sub, pb, ls);
      exp_group<INT4, MASKED, 0, PV_E4M3, 0, 1>(sc, fac, m_sub, pb, ls);
      exp_group<INT4, MASKED, 0, PV_E4M3, 0, 2>(sc, fac, m_sub, pb, ls);
      exp_group<INT4, MASKED, 0, PV_E4M3, 0, 3>(sc, fac, m_sub, pb, ls);
      exp_group<INT4, MASKED, 0, PV_E4M3, 1, 0>(sc, fac, m_sub, pb, ls);
      exp_group<INT4, MASKED, 0, PV_E4M3, 1, 1>(sc, fac, m_sub, pb, ls);
      exp_group<INT4, MASKED, 0, PV_E4M3, 1, 2>(sc, fac, m_sub, pb, ls);
      exp_group<INT4, MASKED, 0, PV_E4M3, 1, 3>(sc, fac, m_sub, pb, ls);
      st.l_run = __fmaf_rn(alpha, st.l_run, ls);
    };
    if (j < n_plain) attend(std::false_type{}); else attend(std::true_type{});
    block_rescale<DW>(st, alpha);
    v4i va[2 * CTW];
#pragma unroll
    for (int i = 0; i < 2 * CTW; ++i) {
      const int ct = w * CTW + i / 2;
      va[i] = s_v[cur][(ct * 2 + (i & 1)) * 64 + (lane ^ ((2 * ct + (n >> 4)) & 7))];
    }
    pv_step<DW, 0, PV_E4M3>(st, va, pb);
    if constexpr (CTW > 1) pv_step<DW, (CTW > 1 ? 1 : 0), PV_E4M3>(st, va, pb);
    if constexpr (CTW > 2) { pv_step<DW, (CTW > 2 ? 2 : 0), PV_E4M3>(st, va, pb); pv_step<DW, (CTW > 2 ? 3 : 0), PV_E4M3>(st, va, pb); }
  }
  if (!col_ok) return;

  float l_tot = st.l_run;
  {
    const unsigned u = __float_as_uint(l_tot);
    const auto sw = __builtin_amdgcn_permlane32_swap(u, u, false, false);
    l_tot = __uint_as_float(sw[0]) + __uint_as_float(sw[1]);
  }
  // Row constant of the log-sum-exp, kappa <q, mean(K)>, for whoever finishes the row.  Added in the order of the quantizers'
  // lanes: runs of CR consecutive channels, then neighbours in pairs, so that the two halves of the wavefront, which take
  // half of the channels each, meet last.  (Here and not beside Q^: the d = 256 4-bit form, which has no register to spare in
  // the loop, then keeps everything in registers: 16 heads, 30000 keys, 249 -> 229 us.)
  float lse_corr = 0.0f;
  if (p.lse && w == 0 && split == 0) {
    constexpr int CR = INT4 ? D / 4 : 8;
    int row = (int)sq.q0 + query;
    asm volatile("" : "+v"(row));          // (the address is formed anew: kept from the start, it would cost the loop registers)
    const unsigned short* qrow = x.q + row_offset(p.om, head_offset(p.om, (unsigned)(bh + hq)), row);
    double runs[D / 2 / CR];
#pragma unroll
    for (int i = 0; i < D / 2 / CR; ++i) {
      runs[i] = 0.0;
#pragma unroll
      for (int e = 0; e < CR; e += 8) {
        const int c = half * (D / 2) + i * CR + e;
        float x8[8];
        unpack8<BF16>(*reinterpret_cast<const uint4*>(qrow + c), x8);
#pragma unroll
        for (int k = 0; k < 8; ++k) runs[i] += (double)x8[k] * (double)s_km[c + k];
      }
    }
    lse_corr = (float)((double)p.kappa * butterfly_sum<32>(pair_sum(runs)));
  }
  if (p.splits > 1) {
    if (p.lse && w == 0 && split == 0 && half == 0) x.q_corr[(bh + hq) * BQ + query] = lse_corr;
    const size_t prow = (size_t)blockIdx.x * BQ + col;
    if (w == 0 && half == 0) { p.part_el[prow * 2] = m_sub; p.part_el[prow * 2 + 1] = l_tot; }
#pragma unroll
    for (int ct = 0; ct < CTW; ++ct) {
#pragma unroll
      for (int g = 0; g < 4; ++g) {
        const v4f o4 = {st.O[ct][4 * g], st.O[ct][4 * g + 1], st.O[ct][4 * g + 2], st.O[ct][4 * g + 3]};
        *reinterpret_cast<v4f*>(p.part_o + prow * D + DW * w + 32 * ct + 8 * g + 4 * half) = o4;
      }
    }
    return;
  }
  if (p.lse && w == 0 && half == 0)
    p.lse[lse_index(p, sq, b, h + hq, query)] = LN2 * ((m_sub + __builtin_amdgcn_logf(l_tot)) + lse_corr);
  const float inv_l = __fdiv_rn(1.0f, l_tot);
  unsigned short* orow = reinterpret_cast<unsigned short*>(p.out) +
                         row_offset(p.om, head_offset(p.om, (unsigned)(bh + hq)), (int)sq.q0 + query);
#pragma unroll
  for (int ct = 0; ct < CTW; ++ct) {
#pragma unroll
    for (int g = 0; g < 4; ++g) {
      const int oc = DW * w + 32 * ct + 8 * g + 4 * half;
      const v4f sc = *reinterpret_cast<const v4f*>(&s_vs[oc]);
      float o4[4];
#pragma unroll
      for (int r = 0; r < 4; ++r) o4[r] = __fmul_rn(__fmul_rn(st.O[ct][4 * g + r], inv_l), sc[r]);
      *reinterpret_cast<uint2*>(orow + oc) = make_uint2(pack16x2<BF16>(o4[0], o4[1]), pack16x2<BF16>(o4[2], o4[3]));
    }
  }
}

// Calls the kernel above serves: the 32 columns of a tile hold all queries that meet a KV head (beyond 32 the softmax piece would be
// repeated for columns that another wavefront holds on the general path), with the default groups, data types and smoothing; in the
// 4-bit mode Delta-S in float64 (the library's own choice for so few block means).  A workgroup works through its chunk block by
// block, 0.7 to 2.8 us each, where the general path spreads the quantizers over the chip: with few workgroups and long chunks that
// serial chain is longer than the launches it saves.  Whole calls whose general path has more than two preprocessing launches, or with
// the statistics supplied, general path / this one, 64 to 104 workgroups: 1.02 to 1.91 at any length (64, chunks of 128 blocks: 1.02
// to 1.21).  4 workgroups, one chunk each: of 12 blocks 1.00 (256 channels, 4-bit) to 1.30, of 20 0.86 (256, 4-bit), 1.00 (128) and
// 1.11 (64), in the 8-bit mode 1.02, 1.16, 1.19; of 32 0.78, 0.87, 0.97 and 0.92, 1.06, 1.07.  With five to eight heads in a group,
// 4-bit: one workgroup of 8 blocks of 256 channels 0.94, 4 of 12 of 128 channels 1.06, of 20 0.90.  16 workgroups: chunks of 20 blocks
// of 256 channels 0.97 (4-bit) and 1.16, of 32 of 128 0.96 and 1.14, of 32 of 64 1.06 and 1.12.  Measured with
// ceil(512 / tiles) chunks: of 8 to 15 blocks until there are 512 workgroups or 64 chunks.  The automatic ones are counted in whole rounds of workgroups
// (chunks_of_few_tiles), so 147 tiles of 300 blocks have three of 100 in 441 workgroups; the two differ only where there are more workgroups than any line
// below, and every call of 1 to 255 tiles and 1 to 1200 blocks goes the same way with either.
// Where the general path has two (small_call) and the statistics are not supplied this kernel came after the statistics and their
// reduction and saved none; these figures are of that form, 2 to 4 us a call before raw_reduces.  4-bit, up to 8 queries, 48 workgroups and more 0.99 to 2.05 at any length; 32 to 47, chunks of up
// to 3 blocks 1.04 to 1.35, of more 0.90 to 1.21; fewer, of 4 blocks of 64 channels 0.99 to 1.08, of 2 of 128 1.01 to 1.15, of 3 of
// 256 1.02 to 1.09, then 0.95 (6 blocks of 64), 0.90 (6 of 128), 0.86 (5 of 256), 0.66 to 0.90 (20 and more).  It adds up the block
// means of more queries one by one: 20 to 32 queries, 48 to 95 workgroups 0.88 to 1.10, fewer 0.72 to 1.00, but 1 or 2 blocks of 256
// channels 1.00 to 1.13.  8-bit, 32 workgroups and more 0.98 to 2.00; 16 to 31, chunks of up to 9 / 6 / 4 blocks 0.98 to 1.70; fewer,
// of 6 blocks of 64 channels 0.99 to 1.04, of 4 of 128 1.01 to 1.17, of 3 of 256 1.13 to 1.23, then 0.97 (10 to 12 of 64), 0.95 (7 of
// 128), 0.83 (12 of 256).
bool attention_raw_ok(const Dims& D) {
  const int G = D.H / D.Hkv;
  const long long groups = (long long)D.B * D.Hkv * D.splits;
  const int chunk = (D.nKb + D.splits - 1) / D.splits;
  int longest = D.int4 ? (G <= 4 ? 4 : 0) + 1024 / D.d : 8 + 1536 / D.d;
  if (groups >= 16) longest += longest / 2;
  int many = 64;
  if (small_call(D) && !D.stats_given) {
    if (!D.int4) { longest = D.d == 64 ? 6 : (D.d == 128 ? 4 : 3); if (groups >= 16) longest += longest / 2; many = 32; }
    else if (D.N <= 8) { longest = D.d == 64 ? 4 : (D.d == 128 ? 2 : 3); many = 48; }
    else { longest = D.d == 256 ? 2 : 0; many = 96; }
  }
  return G <= PACK_G && (long long)G * D.N <= 32 && (groups >= many || chunk <= longest) && D.kg == KGROUP && !D.block_groups && D.pvf == PV_E4M3 &&
         D.smooth_k && D.smooth_q && !D.smooth_v && (!D.int4 || D.ds_mode == 2);
}

// Whether the kernel reduces the partial results of the statistics pass itself (every workgroup for its head) instead of a launch of its
// own in front.  The launch is 2 to 4 us of a call, the reduction reads 12 bytes a channel and 256-key chunk in every workgroup.  Whole calls on
// inputs in turn, this / a launch: 100 keys 0.82 to 0.84, 300 0.88 to 0.92, 500 to 1000 0.89 to 0.97, 2000 0.88 to 0.97, 8000 of 128 channels
// 0.94 (8 KV heads) to 0.99 (64), 32000 0.97 to 0.98, 60000 of 64 channels 0.96 to 0.97, of 128 1.01; 8000 of 256 channels 0.98, 12000 and
// more 1.01 to 1.03; past the 256 MB of the memory-side cache, where the partial results lie, 0.98 to 1.01.
bool raw_reduces(const Dims& D) {
  const int nchunk = (D.Nk + STAT_ROWS - 1) / STAT_ROWS;
  return !D.stats_given && nchunk * D.d <= (D.d == 256 ? 8192 : 16384) && 4LL * D.B * D.Hkv * D.Nk * D.d <= 256LL << 20;
}

template <int DD, bool INT4, bool CAUSAL>
static hipError_t launch_raw_t(const Dims& D, const Ptrs& P, hipStream_t s) {
  AttnParams p = attn_params(D, P);
  p.total_tiles = D.B * D.Hkv;
  RawParams x;
  x.q = (const unsigned short*)P.q; x.k = (const unsigned short*)P.k; x.v = (const unsigned short*)P.v;
  x.k_mean = P.k_mean; x.q_corr = P.q_corr;
  x.k_sum = raw_reduces(D) ? P.k_sum : nullptr; x.v_max = P.v_max; x.v_scale = P.v_scale; x.nchunk = (D.Nk + STAT_ROWS - 1) / STAT_ROWS;
  x.km = make_tensor_map(D.nhd, D.Hkv, D.Nk, D.d, D.seq.cu_q != nullptr);
  const int grid = p.total_tiles * D.splits;
  const bool many = INT4 && D.H / D.Hkv > 4;
  if constexpr (INT4) {
    if (D.N == 1) {                // (of a packed batch: the longest sequence's; without a mask: one query sees every key)
#define SAGE_RAW_LONE(BF, HEADS) k_attn_raw<DD, true, false, BF, HEADS, true><<<grid, RAW_THREADS, 0, s>>>(p, x)
      if (D.bf16) { if (many) SAGE_RAW_LONE(true, PACK_G); else SAGE_RAW_LONE(true, 4); }
      else        { if (many) SAGE_RAW_LONE(false, PACK_G); else SAGE_RAW_LONE(false, 4); }
#undef SAGE_RAW_LONE
      return D.splits > 1 ? launch_merge_packed(D, p, s) : hipGetLastError();
    }
  }
#define SAGE_RAW_LAUNCH(BF) \
  do { \
    if (many) k_attn_raw<DD, INT4, CAUSAL, BF, INT4 ? PACK_G : 4><<<grid, RAW_THREADS, 0, s>>>(p, x); \
    else k_attn_raw<DD, INT4, CAUSAL, BF, 4><<<grid, RAW_THREADS, 0, s>>>(p, x); \
  } while (0)
  if (D.bf16) SAGE_RAW_LAUNCH(true); else SAGE_RAW_LAUNCH(false);
#undef SAGE_RAW_LAUNCH
  if (D.splits > 1) return launch_merge_packed(D, p, s);
  return hipGetLastError();
}

hipError_t launch_attention_raw(const Dims& D, const Ptrs& P, hipStream_t s) {
#define SAGE_RAW(DD) \
  do { \
    if (D.int4) return D.causal ? launch_raw_t<DD, true, true>(D, P, s) : launch_raw_t<DD, true, false>(D, P, s); \
    return D.causal ? launch_raw_t<DD, false, true>(D, P, s) : launch_raw_t<DD, false, false>(D, P, s); \
  } while (0)
  if (D.d == 256) SAGE_RAW(256);
  else if (D.d == 128) SAGE_RAW(128);
  else SAGE_RAW(64);
#undef SAGE_RAW
}

}  // namespace sage
