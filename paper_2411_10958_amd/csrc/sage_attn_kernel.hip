// Fused quantized attention kernel for gfx950: the inner loop and epilogue of the paper's
// Algorithm 1.  One workgroup (4 wavefronts) owns one 128-query smoothing block of one
// (batch, head); each wavefront owns 32 queries and walks the 64-key blocks.
//
// The score tile is computed transposed, S^T = K^ Q^^T, with 32x32 MFMAs (v_mfma_i32_32x32x32_i8 in
// the 8-bit mode, the FP6 operand format of v_mfma_f32_32x32x64_f8f6f4 in the 4-bit mode): rows are
// keys, columns are queries, so a lane holds ONE query (column lane%32) and, thanks to the row
// permutation baked into the packed K^ layout, 16 consecutive keys per 32-key tile.  Row max
// and row sum are therefore lane-local plus one exchange between the two lane halves, one
// lane needs one delta_Q and one delta_K per tile (Sec. 3.2's per-thread principle on this
// accumulator layout; finer key scales are a template option), and the FP8 P~ registers are directly the B operand of
// O^T = V^^T P~^T (v_mfma_f32_32x32x64_f8f6f4, K = 64 = one accumulation block).  The
// instruction sums the block's 64 products internally (level 1 of Sec. 3.4) and adds its C
// operand - the running O - in full FP32 (level 2).
#include "sage_attn_core.h"

namespace sage {

// Blocks left at which a workgroup of the last round lowers its priority for the (i + 1)-th time (in the kernel): the last step is what
// two of them may end apart.
template <int D> __device__ constexpr int tail_left(int i) { return D == 64 ? (i == 0 ? 40 : i == 1 ? 20 : 8) : (i == 0 ? 28 : i == 1 ? 12 : 4); }
__device__ __forceinline__ void set_priority(int p) {     // (the instruction takes a constant)
  if (p == 3) __builtin_amdgcn_s_setprio(3);
  else if (p == 2) __builtin_amdgcn_s_setprio(2);
  else if (p == 1) __builtin_amdgcn_s_setprio(1);
  else __builtin_amdgcn_s_setprio(0);
}

// PACK (with SPLIT; short queries, grouped KV heads): a tile holds ALL queries of the G = H / H_kv query heads that
// share one KV head - column c of the tile is query c % n of head c / n of the group, n the sequence's query count
// (G N <= 128 for the longest sequence, G <= PACK_G) - so
// the KV head's codes are walked once for the whole group instead of once per query head with 128 - N idle columns
// each.  Everything that belongs to a query (its codes, scale, Delta-S row, output row) is then looked up per lane.
template <int D, bool INT4, bool CAUSAL, bool BF16, int GM, int PVF, bool SPLIT = false, bool PACK = false>
__global__ void __launch_bounds__(256, (attn_occupancy<D, GM, PVF>())) k_attn_fwd(const AttnParams p) {
  constexpr bool OCC3 = attn_occupancy<D, GM, PVF>() >= (D == 256 ? 2 : 3);     // the form without a software pipeline
  static_assert(!PACK || (SPLIT && OCC3 && GM == 0), "packed tiles come with the split key range and the default groups");
  constexpr int DSR = PACK && INT4 ? PACK_G : 1;   // Delta-S rows per stage
  constexpr int KSC = GM == 0 ? 4 : (GM == 1 ? 16 : 64);    // key scales per block
  constexpr int QG = GM == 0 ? QGROUP : 1;                  // queries per scale
  constexpr int CT = D / 32;          // 32-channel tiles of the output
  constexpr int KC = D * BKV / 16;    // 16-byte chunks of one V^ block
  constexpr int KCK = (int)(k_block_bytes(D, INT4) / 16);   // 16-byte chunks of one K^ block
  constexpr int CPT = KC / 256;       // V^ chunks per thread per block copy (2 or 1)
  // LDS stages: block j is read while j+1 and j+2 arrive (d = 256 without the software pipeline: two stages of
  // 29 KB, so that two workgroups fit a CU)
  constexpr int NST = (D == 256 && attn_occupancy<D, GM, PVF>() >= 2) ? 2 : 3;
  constexpr int PD = NST - 1;         // copies run this many blocks ahead
  constexpr int XC = 16 * DSR + 16;   // chunks of the small part: DSR rows of 64 Delta-S floats, then up to 64 key scales
  constexpr int STAGE = KCK + KC + XC;   // chunks per stage: K^, V^, small part
  __shared__ v4i lds[NST][STAGE];
  __shared__ __align__(16) float s_vs[2][D];   // delta_V and (smooth-V option) mean(V) of this KV head, for the epilogue

  // XCD-aware tile order: consecutive workgroup ids land on different XCDs (8 of them), so
  // give every XCD a contiguous range of tiles - tiles of one head then share one L2.
  // Under a causal mask a tile's work grows with its position, and workgroups start in index order.  There the
  // heads are taken in groups of 32 and a group's tiles are issued heaviest first ACROSS its heads (all their last
  // tiles, then all their last but one, ...), workgroup i taking the i-th tile of that list: every XCD then gets
  // every eighth tile of each weight - an equal share of the work whatever the head count - and, with 32 heads in a
  // group, the tiles of the same four heads.  Head by head the heavy tiles of an XCD's last head would start late
  // and finish long after the rest (13 % of the kernel's time at N = 8192, 1.5 % at N = 16384), and contiguous
  // ranges that do not hold whole heads (a head count that 8 does not divide) differ in work by up to a factor of
  // three.  More than four heads per XCD at a time no longer share its L2 once a head's codes exceed about 2 MB
  // (16 interleaved heads of 16384 keys ran 13 % slower than four; up to 4096 keys 16 are 4 % faster than four).
  // Sequences beyond 16384 tokens take groups of 8 heads - one head per XCD at a time, heaviest tile first: four
  // interleaved heads no longer share an XCD's L2 there (N = 32768: 1.5 % slower), and the equal shares still
  // count when 8 does not divide the head count (28 heads of 32768 tokens: +4.5 %).
  // A packed batch: sequence by sequence, a long one late in the batch would start its heavy tiles when the short ones are
  // nearly done, and in contiguous ranges (no mask) each XCD would work on sequences of its own.  The tiles of a ragged one
  // (packed_in_bands) go out in bands of BAND_LEVELS positions instead, from the last position of the longest sequence down, in a band
  // sequence by sequence, heaviest first - so that the tiles of a head still run close together.
  const int n_wg = SPLIT ? p.total_tiles * p.splits : p.total_tiles;
  const int per_xcd = (n_wg + 7) / 8;
  const int in_xcd = blockIdx.x / 8;
  int tile = (blockIdx.x % 8) * per_xcd + in_xcd;
  int split = 0;
  int bh, qb;
  const bool bands = !SPLIT && p.seq.cu_q && packed_in_bands(CAUSAL, p.seq.cu_q[p.B] - p.seq.cu_q[0], p.B, p.N);
  if (!SPLIT && (CAUSAL || bands)) {
    tile = blockIdx.x;
    if (tile >= n_wg) return;
    const int BH = p.total_tiles / p.nQb;
    const int GS = bands ? p.H : p.nQb <= 32 ? 128 : (p.nQb <= 128 ? 32 : 8);  // heads per group
    int in_band = tile, q_top = p.nQb - 1, levels = p.nQb;      // this band's tiles: positions q_top, q_top - 1, ... of every head
    if (bands) {
      const int band = tile / (BAND_LEVELS * BH);
      in_band = tile - band * BAND_LEVELS * BH;
      q_top -= band * BAND_LEVELS;
      levels = min(BAND_LEVELS, q_top + 1);
    }
    const int full = BH / GS;                                   // groups of GS heads; the last one may be smaller
    int grp = in_band / (GS * levels), g = GS;
    if (grp >= full) { grp = full; g = BH - full * GS; }
    const int within = in_band - grp * GS * levels;
    bh = grp * GS + within % g;
    qb = q_top - within / g;
  } else {
    if (tile >= n_wg) return;
    if constexpr (SPLIT) { split = tile % p.splits; tile /= p.splits; }
    bh = tile / p.nQb;
    qb = CAUSAL ? p.nQb - 1 - tile % p.nQb : tile % p.nQb;   // heavy tiles first
  }
  if (tile >= p.total_tiles) return;
  // PACK: tiles count (batch, KV head) pairs; bh is the first query head of the tile's group
  if constexpr (PACK) bh = (tile / p.Hkv) * p.H + (tile % p.Hkv) * (p.H / p.Hkv);
  const int b = bh / p.H, h = bh % p.H;
  const size_t bhkv = (size_t)b * p.Hkv + h / (p.H / p.Hkv);
  // this sequence's lengths (the launch's N, Nk unless the batch is a variable-length one; slab
  // strides below keep the block counts of the longest sequence)
  const Seq sq = seq_of(p.seq, (unsigned)b, p.N, p.Nk);
  if (qb * BQ >= sq.n) return;                 // a tile past the end of a shorter sequence

  const int t = threadIdx.x, lane = t & 63;
  if (sq.nk == 0) {                            // no keys at all: the rows are defined as zeros
    if (SPLIT && split != 0) return;           // (written once; the merge kernel leaves such a tile alone)
    for (int g = 0; g < (PACK ? p.H / p.Hkv : 1); ++g) {        // (PACK: the tile's rows belong to the whole group)
      unsigned short* o = reinterpret_cast<unsigned short*>(p.out) + head_offset(p.om, (unsigned)(bh + g));
      for (int idx = t; idx < BQ * (D / 8); idx += 256) {
        const int row = qb * BQ + idx / (D / 8);
        if (row < sq.n)
          *reinterpret_cast<uint4*>(o + row_offset(p.om, 0, (int)sq.q0 + row) + (idx % (D / 8)) * 8) =
              make_uint4(0u, 0u, 0u, 0u);
      }
      if (p.lse && t < BQ && qb * BQ + t < sq.n) p.lse[lse_index(p, sq, b, h + g, qb * BQ + t)] = -INFINITY;
    }
    return;
  }
  const int w = __builtin_amdgcn_readfirstlane(t >> 6);
  const int n = lane & 31, half = lane >> 5;
  // PACK: column w * 32 + n of the tile is query qi of head bh + hq; columns past the group's G N queries work on
  // query 0 of the first head and write nothing
  int hq = 0, qi = 0;
  bool col_ok = true;
  if constexpr (PACK) {
    const int col = w * WQ + n;
    col_ok = col < (p.H / p.Hkv) * sq.n;      // (sq.n >= 1 here)
    hq = col_ok ? col / sq.n : 0;
    qi = col_ok ? col - hq * sq.n : 0;
  }
  const int q_lo = PACK ? 0 : qb * BQ + w * WQ;          // first query of this wavefront
  const int q_hi = PACK ? sq.n - 1 : q_lo + WQ - 1;      // ... and the last
  const int query = PACK ? qi : q_lo + n;
  const size_t bhq = (size_t)bh + hq;                    // this lane's query head

  const v4i* gk = reinterpret_cast<const v4i*>(p.k_codes + bhkv * (size_t)p.nKb * k_block_bytes(D, INT4));
  const v4i* gv = reinterpret_cast<const v4i*>(p.v_codes + bhkv * (size_t)p.nKb * BKV * D);
  const float* gd = INT4 ? p.delta_s + ((size_t)bh * p.nQb + qb) * p.nKb * BKV : nullptr;
  const float* gs = p.k_scale + bhkv * (size_t)p.nKb * KSC;

  int nblk = (sq.nk + BKV - 1) / BKV;
  if (CAUSAL) nblk = min(nblk, (qb * BQ + BQ - 1 + sq.coff) / BKV + 1);
  int j_begin = 0;                             // this workgroup's key blocks: [j_begin, nblk)
  if constexpr (SPLIT) {
    const int n_vis = CAUSAL ? min(nblk, (qb * BQ + sq.coff) / BKV + 1) : nblk;
    const KeyChunk kc = key_chunk(split, p.splits, nblk, n_vis);
    j_begin = kc.j0;
    nblk = kc.j1;
    if (j_begin >= nblk) {                     // an empty chunk: offset -inf, sum 0 (the merge skips it)
      if (t < BQ) {
        float* el = p.part_el + ((size_t)((PACK ? tile : bh * p.nQb + qb) * p.splits + split) * BQ + t) * 2;
        el[0] = -INFINITY; el[1] = 0.0f;
      }
      return;
    }
  }

  // Block copies, in pieces of 64 chunks (1 KB, one copy instruction): whole rounds of four K^ and V^ pieces, one per
  // wavefront, then what is left - K^ pieces, the Delta-S row, the key scales - as a round of one "rest" piece per
  // wavefront, fewer lanes where it is shorter (and a single piece by one wavefront where that leaves one over).
  // Which rest piece a wavefront has is settled here, once per tile, so the loop has no branches by wavefront: the
  // copies bound it beside the vector issue (without them it takes 11 % less at 128 channels, 16 % at 256).  Against a
  // branch per piece: 256 channels, 16 heads of 8192 tokens, causal 261 -> 249 us (4-bit mode; its spilled registers
  // went as well) and 298 -> 293 (8-bit), 128 channels, 128 heads of 4096 tokens, 4-bit 575 -> 565; 64 channels and the
  // 8-bit mode at 128, which had one branch less to lose, the same.
  const unsigned lds0 = (unsigned)(size_t)(__attribute__((address_space(3))) char*)&lds[0][0];
  constexpr int KG = KCK / 64, KR = KG / 4, KL = KG % 4;
  constexpr int NREST = KL + (INT4 ? 1 : 0) + 1;            // K^ pieces, Delta-S, scales
  constexpr bool REST = !PACK && NREST >= 2;                // a round of rest pieces (packed tiles: several Delta-S rows)
  constexpr int SC_W = NREST - 1;                           // the rest piece that holds the scales
  const char* rest_p = nullptr;
  unsigned rest_step = 0, rest_lds = 0, rest_lanes = 0;
  if constexpr (REST) {
    const char* pk = reinterpret_cast<const char*>(gk + (KR * 4 + w) * 64);
    if (w < KL) {
      rest_p = pk; rest_step = KCK * 16; rest_lds = (KR * 4 + w) * 1024; rest_lanes = 64;
    } else if (INT4 && w == KL) {
      rest_p = reinterpret_cast<const char*>(gd); rest_step = BKV * 4; rest_lds = (KCK + KC) * 16; rest_lanes = 16;
    } else if (w == SC_W) {
      rest_p = reinterpret_cast<const char*>(gs); rest_step = KSC * 4; rest_lds = (KCK + KC) * 16 + 256; rest_lanes = KSC / 4;
    }
    rest_p = uniform_ptr(rest_p);
    rest_step = __builtin_amdgcn_readfirstlane(rest_step);
    rest_lds = __builtin_amdgcn_readfirstlane(rest_lds);
    rest_lanes = __builtin_amdgcn_readfirstlane(rest_lanes);
  }
  const unsigned long long rest_mask = rest_lanes == 64 ? ~0ull : (1ull << rest_lanes) - 1;
  auto issue = [&](int j, int st) {
    const unsigned sb = lds0 + (unsigned)st * (STAGE * 16);
    const unsigned v16 = (unsigned)lane * 16;
    const char* k0 = reinterpret_cast<const char*>(gk) + (size_t)j * (KCK * 16) + w * 1024;
    const char* v0 = reinterpret_cast<const char*>(gv) + (size_t)j * (KC * 16) + w * 1024;
#pragma unroll
    for (int i = 0; i < KR; ++i) dma_b128(k0 + i * 4096, v16, sb + w * 1024 + i * 4096);
#pragma unroll
    for (int i = 0; i < CPT; ++i) dma_b128(v0 + i * 4096, v16, sb + KCK * 16 + w * 1024 + i * 4096);
    if constexpr (REST) dma_b128_lanes(rest_p + (size_t)j * rest_step, v16, sb + rest_lds, rest_mask);
    if constexpr (PACK) {
      if constexpr (KL > 0) { if (w < KL) dma_b128(k0 + KR * 4096, v16, sb + w * 1024 + KR * 4096); }
      if (INT4 && w == 2) {            // one Delta-S row per query head of the group (consecutive heads, one row each)
        const int G = p.H / p.Hkv;
        for (int g = 0; g < G; ++g)
          dma_b32(gd + (size_t)g * p.nKb * BKV + (size_t)j * BKV, (unsigned)lane * 4, sb + (KCK + KC) * 16 + 256u * g);
      }
    }
    if constexpr (!REST || NREST > 4) {
      if (w == 3 && lane < KSC) dma_b32(gs + (size_t)j * KSC, (unsigned)lane * 4, sb + (KCK + KC) * 16 + 256 * DSR);
    }
  };
  // Every wavefront issues at least MINC copies per block, in block order, and loads complete in
  // order: "at most MINC outstanding" therefore means every block but the newest has landed.  (A copy of no lanes may not
  // count as outstanding: a form that waits by number - causal, with the software pipeline - has a rest piece for every wavefront.)
  constexpr int MINC = KR + CPT + (REST ? 1 : 0);
  static_assert(OCC3 || !CAUSAL || !REST || NREST >= 4, "a wavefront without a rest piece does not issue MINC copies");
  auto wait_all_but_newest = [&]() {
    static_assert(MINC >= 1 && MINC <= 12, "copy count per block");
    asm volatile("s_waitcnt vmcnt(%0) lgkmcnt(0)" :: "n"(MINC) : "memory");
  };
  auto wait_all = [&]() { asm volatile("s_waitcnt vmcnt(0) lgkmcnt(0)" ::: "memory"); };

  // Without a causal mask the copies of the first two blocks go out before anything else of the tile is
  // requested, so that their round trip and that of the Q^ loads below overlap (1.2 % on N = 4096; copies
  // older than the compiler's own loads are harmless to its wait counts: loads complete in order, so
  // "at most n outstanding" still covers the load it means).  Under a causal mask, where many tiles are
  // short, the same order measured 1 % slower at N = 8192 and 16384, so there the copies follow the loads.
  constexpr bool COPIES_FIRST = !CAUSAL;
  // The epilogue's per-channel constants travel to LDS now (wavefronts 2 and 3, one copy per 64 channels):
  // read from global memory at the end of the tile, their round trip was idle time of the workgroup's share
  // of the CU.  These copies are older than every block copy, so the wait counts below still hold.
  {
    const unsigned vs0 = (unsigned)(size_t)(__attribute__((address_space(3))) char*)&s_vs[0][0];
    if (w == 2) {
#pragma unroll
      for (int i = 0; i < D / 64; ++i) dma_b32(p.v_scale + bhkv * D + 64 * i, (unsigned)lane * 4, vs0 + 256u * i);
    } else if (w == 3 && p.v_mean) {
#pragma unroll
      for (int i = 0; i < D / 64; ++i) dma_b32(p.v_mean + bhkv * D + 64 * i, (unsigned)lane * 4, vs0 + 4u * D + 256u * i);
    }
  }
  if constexpr (COPIES_FIRST) {
    issue(j_begin, 0);
    if (PD > 1 && j_begin + 1 < nblk) issue(j_begin + 1, 1);
  }

  // ---- this wavefront's Q^ operands (registers, for the whole kernel) and scale ----
  typedef typename QkOperand<INT4>::type qk_op;
  constexpr int NP = qk_pieces<D, INT4>();
  qk_op qreg[NP];
  {
    // (PACK: the lane's query sits in 32-query slice qi / 32 of its own head's slab, at lane position qi % 32)
    const int slice = PACK ? qi / WQ : w;
    const int pos = PACK ? (qi % WQ) + 32 * half : lane;
    const v4i* gq = reinterpret_cast<const v4i*>(p.q_codes + (bhq * p.nQb + qb) * q_slab_bytes(D, INT4)) +
                    (size_t)slice * (q_slab_bytes(D, INT4) / 16 / (BQ / WQ));
#pragma unroll
    for (int s = 0; s < NP; ++s) qreg[s] = load_qk_operand<INT4>(gq, s, pos);
  }
  const int row_in_block = PACK ? qi : w * WQ + n;       // the query's place in its smoothing block
  const float dq = p.q_scale[(bhq * p.nQb + qb) * (BQ / QG) + row_in_block / QG];
  // the row constant of the log-sum-exp output, fetched now so that the epilogue does not wait for it
  float lse_corr = 0.0f;
  if (p.lse) lse_corr = p.q_corr[(bhq * p.nQb + qb) * BQ + row_in_block];

  RowState<D> st;
#pragma unroll
  for (int ct = 0; ct < CT; ++ct) {
#pragma unroll
    for (int v = 0; v < 16; ++v) st.O[ct][v] = 0.0f;
  }
  st.m_run = -INFINITY;
  st.l_run = 0.0f;

  // The wavefront walks all nblk blocks of the workgroup (copies and barriers are shared):
  // blocks [0, n_act) hold keys visible to some of its queries, of which [0, n_plain) need no
  // mask; past n_act (causal only) it just helps with the copies.
  int n_plain = min(nblk, sq.nk / BKV);                        // blocks without padded keys
  int n_act = nblk;                                            // blocks with any visible key
  if (CAUSAL) {
    n_plain = min(n_plain, (q_lo + sq.coff + 1) / BKV);        // key0 + 63 <= q_lo + coff
    n_act = min(nblk, (q_hi + sq.coff) / BKV + 1);             // key0 <= q_hi + coff
  }
  if constexpr (PACK) {
    // a wavefront whose 32 columns all lie past the group's queries only keeps up the copies and the barriers
    if (w * WQ >= (p.H / p.Hkv) * sq.n) n_plain = n_act = j_begin;
  }
  n_plain = __builtin_amdgcn_readfirstlane(n_plain);
  n_act = __builtin_amdgcn_readfirstlane(n_act);

  // Keys from here on are masked like the padding past the sequence's end.  For a chunk of a split key range that
  // is the chunk's end: the pipeline always forms the scores of one block past the last (from a stale stage), and
  // its running-max update must see them masked, or the exponent offset handed to the merge would not be the one
  // the sums were taken under.
  const int n_keys_end = SPLIT ? min(sq.nk, nblk * BKV) : sq.nk;

  // Software pipeline, one barrier per block, three LDS stages; every MFMA is issued between
  // pieces of vector work that do not depend on it, one at a time (a burst of MFMAs would hold up
  // the wavefront's own vector instructions behind it).  On entry to iteration j the dequantized
  // scores of block j (`sc`), their alpha and exponent offset are in registers, stage j%3 holds
  // block j and the copy of block j+1 is in flight.  The iteration
  //   B. waits for its own share of block j+1 and meets the other wavefronts at the barrier:
  //      block j+1 is visible, and nobody reads block j-1's stage any more,
  //   C. starts the LDS reads of K^_{j+1} and the copy of block j+2 into block j-1's stage,
  //   R. rescales O if a running max moved (covers the latency of C's reads),
  //   X. exponentials, row sum and FP8 codes of block j, four keys at a time, with one score MFMA
  //      of block j+1 issued in front of each piece; half way, the LDS reads of V^_j, of block j+1's scales
  //      and of the first key tile's half of its Delta-S row are started - the latter straight into the score
  //      registers that half of the exponentials has just finished with; the other half follows at the end,
  //   Y. the P~V MFMAs of block j, each followed by a piece of block j+1's dequantization, then
  //      block j+1's running-max update.
  // Past the wavefront's last block C, X and Y work on a stale stage (in bounds, results unused):
  // unconditional, so that no register stays live for the sake of a path not taken.
  qk_op ka[2 * NP];
  v4i va[2 * CT];
  KeyScales<GM> ks;
  v16i raw[2], sc[2];                 // raw scores being produced / dequantized scores of block j
  auto read_k = [&](int stg) {
    read_k_block<D, INT4>(&lds[stg][0], lane, ka);
  };
  auto read_v = [&](int stg) {
#pragma unroll
    for (int i = 0; i < 2 * CT; ++i) va[i] = lds[stg][KCK + i * 64 + lane];
  };
  // With a scale per key in the 8-bit mode the block's 32 factors stay live through the exponentials (they are
  // fused into the exponent's argument), so the next block's 32 key scales are fetched after them, not half way.
  constexpr bool LATE_SCALES = GM == 2 && !INT4;
  // Delta-S of key tile kt of the block in stage stg, into the registers the tile's scores will be formed in
  // (they are free once the previous block's exponentials of that tile are done)
  auto read_ds = [&](int stg, int kt) {
    if constexpr (INT4) {
      const v4f* dsv = reinterpret_cast<const v4f*>(reinterpret_cast<const float*>(&lds[stg][KCK + KC]) + 64 * hq + 32 * kt + 16 * half);
#pragma unroll
      for (int g = 0; g < 4; ++g) {
        const v4f t4 = dsv[g];
#pragma unroll
        for (int r = 0; r < 4; ++r) sc[kt][4 * g + r] = __float_as_int(t4[r]);
      }
    }
  };
  auto read_scales = [&](int stg) {
    const float* lx = reinterpret_cast<const float*>(&lds[stg][KCK + KC]) + 64 * (DSR - 1);
    if constexpr (GM == 0) {
      ks.s[0] = lx[64 + half];
      ks.s[1] = lx[66 + half];
    } else if constexpr (GM == 1) {
      ks.s[0] = *reinterpret_cast<const v4f*>(lx + 64 + 4 * half);
      ks.s[1] = *reinterpret_cast<const v4f*>(lx + 72 + 4 * half);
    } else {
#pragma unroll
      for (int kt = 0; kt < 2; ++kt) {
        const v4f* kv = reinterpret_cast<const v4f*>(lx + 64 + 32 * kt + 16 * half);
#pragma unroll
        for (int g = 0; g < 4; ++g) ks.s[kt][g] = kv[g];
      }
    }
  };
  // The compiler does not see the copies, and it would otherwise leave its waits for the ordinary
  // loads of Q^ and the scale inside the loop, where they would also wait for the copies then in
  // flight: use those registers here so that the loads are complete before the loop.
#pragma unroll
  for (int s = 0; s < NP; ++s) {
#pragma unroll
    for (int i = 0; i < (int)(sizeof(qk_op) / 4); ++i) use_now(qreg[s][i]);
  }
  use_now(dq);
  use_now(lse_corr);
  if constexpr (COPIES_FIRST) {
    if constexpr (!OCC3) wait_all();
  } else {
    issue(j_begin, 0);
    if (PD > 1 && j_begin + 1 < nblk) { issue(j_begin + 1, 1); if constexpr (!OCC3) wait_all_but_newest(); } else { if constexpr (!OCC3) wait_all(); }
  }
  float alpha, m_sub = -INFINITY;     // of block j (m_sub: nothing summed yet)
  Factors<GM> fj;                     // block j's dequantization factors (used again by the fused exponent)
  constexpr int NQK = qk_steps<D, INT4>();
  constexpr int QPX = NQK > 8 ? 2 : 1;   // score MFMAs issued in front of each of the 8 pieces of the exponentials
  static_assert(NQK <= 16, "score MFMAs per block");
  constexpr int GPC = CT >= 8 ? 1 : 8 / CT;   // dequantization groups per P~V MFMA

#define SAGE_DEQ(MASKED_, GI_, KEY0_)                                                                \
  dequant_group<INT4, CAUSAL, MASKED_, GM, (GI_) / 4, (GI_) % 4>(raw, sc, fn, half, KEY0_,               \
                                                                 query + sq.coff, n_keys_end)
#define SAGE_DEQ_ALL(MASKED_, KEY0_)                                                                 \
  do {                                                                                               \
    SAGE_DEQ(MASKED_, 0, KEY0_); SAGE_DEQ(MASKED_, 1, KEY0_); SAGE_DEQ(MASKED_, 2, KEY0_);           \
    SAGE_DEQ(MASKED_, 3, KEY0_); SAGE_DEQ(MASKED_, 4, KEY0_); SAGE_DEQ(MASKED_, 5, KEY0_);           \
    SAGE_DEQ(MASKED_, 6, KEY0_); SAGE_DEQ(MASKED_, 7, KEY0_);                                        \
  } while (0)
  if constexpr (!OCC3) {
    __syncthreads();
    read_k(0);
    read_ds(0, 0);
    read_ds(0, 1);
    read_scales(0);
    qk_tile<D, INT4>(ka, qreg, raw);    // the first block holds a visible key for every query
    Factors<GM> fn;
    fn.set(dq, p.kappa, ks);
    if (j_begin < n_plain) SAGE_DEQ_ALL(false, j_begin * BKV); else SAGE_DEQ_ALL(true, j_begin * BKV);
    alpha = update_max<D, INT4, GM, PVF>(st, sc, fn, m_sub);
    fj = fn;
  }

  int cur = 0;   // stage of block j
#define SAGE_X(GI_, MASKED_)                                                                         \
  do {                                                                                               \
    if constexpr (QPX == 2) {                                                                        \
      qk_step<D, INT4, 2 * (GI_) < NQK ? 2 * (GI_) : 0>(ka, qreg, raw);                               \
      qk_step<D, INT4, 2 * (GI_) + 1 < NQK ? 2 * (GI_) + 1 : 0>(ka, qreg, raw);                       \
    } else if constexpr ((GI_) < NQK) {                                                              \
      qk_step<D, INT4, (GI_) < NQK ? (GI_) : 0>(ka, qreg, raw);                                      \
    }                                                                                                \
    exp_group<INT4, MASKED_, GM, PVF, (GI_) / 4, (GI_) % 4>(sc, fj, m_sub, pb, ls);                  \
    __builtin_amdgcn_sched_barrier(0);                                                               \
  } while (0)
#define SAGE_Y(CT_, MASKED_)                                                                         \
  do {                                                                                               \
    if constexpr ((CT_) < CT) {                                                                      \
      pv_step<D, (CT_) < CT ? (CT_) : 0, PVF>(st, va, pb);                                           \
      SAGE_DEQ(MASKED_, ((CT_) * GPC) % 8, (j + 1) * BKV);                                           \
      if constexpr (GPC >= 2) SAGE_DEQ(MASKED_, ((CT_) * GPC + 1) % 8, (j + 1) * BKV);               \
      if constexpr (GPC == 4) {                                                                      \
        SAGE_DEQ(MASKED_, ((CT_) * GPC + 2) % 8, (j + 1) * BKV);                                     \
        SAGE_DEQ(MASKED_, ((CT_) * GPC + 3) % 8, (j + 1) * BKV);                                     \
      }                                                                                              \
      __builtin_amdgcn_sched_barrier(0);                                                             \
    }                                                                                                \
  } while (0)
#define SAGE_BODY(MASKED_, MASKED_NEXT_)                                                                    \
  do {                                                                                               \
    const int nx1 = cur == NST - 1 ? 0 : cur + 1;                                                    \
    const int nx2 = nx1 == NST - 1 ? 0 : nx1 + 1;                                                    \
    wait_all();                                                                               /* B */ \
    __syncthreads();                                                                                 \
    read_k(nx1);                                                                              /* C */ \
    if (j + 2 < nblk) issue(j + 2, nx2);                                                             \
    block_rescale<D>(st, alpha);                                                              /* R */ \
    __builtin_amdgcn_sched_barrier(0);                                                               \
    v8i pb;                                                                                          \
    float ls = 0.0f;                                                                                 \
    SAGE_X(0, MASKED_); SAGE_X(1, MASKED_); SAGE_X(2, MASKED_); SAGE_X(3, MASKED_);           /* X */ \
    read_v(cur);                                                                                     \
    read_ds(nx1, 0);                                                                                 \
    if constexpr (!LATE_SCALES) read_scales(nx1);                                                    \
    __builtin_amdgcn_sched_barrier(0);                                                               \
    SAGE_X(4, MASKED_); SAGE_X(5, MASKED_); SAGE_X(6, MASKED_); SAGE_X(7, MASKED_);                  \
    read_ds(nx1, 1);                                                                                 \
    if constexpr (LATE_SCALES) read_scales(nx1);                                                     \
    st.l_run = __fmaf_rn(alpha, st.l_run, ls);                                                       \
    Factors<GM> fn;                                                                                  \
    fn.set(dq, p.kappa, ks);                                                                         \
    SAGE_Y(0, MASKED_NEXT_); SAGE_Y(1, MASKED_NEXT_); SAGE_Y(2, MASKED_NEXT_); SAGE_Y(3, MASKED_NEXT_); /* Y */ \
    SAGE_Y(4, MASKED_NEXT_); SAGE_Y(5, MASKED_NEXT_); SAGE_Y(6, MASKED_NEXT_); SAGE_Y(7, MASKED_NEXT_);         \
    alpha = update_max<D, INT4, GM, PVF>(st, sc, fn, m_sub);                                              \
    fj = fn;                                                                                         \
    cur = nx1;                                                                                       \
  } while (0)
  // Variant for three wavefronts per SIMD (168 registers): no software pipeline inside a wavefront - block j's score
  // product, softmax piece and P~V product run one after the other, and the two other wavefronts of the SIMD fill
  // the waits - so only one block's scores are live at a time.
#define SAGE_E3(GI_, MASKED_) exp_group<INT4, MASKED_, GM, PVF, (GI_) / 4, (GI_) % 4>(sc, fn, m_sub, pb, ls)
#define SAGE_P3(CT_) do { if constexpr ((CT_) < CT) pv_step<D, (CT_) < CT ? (CT_) : 0, PVF>(st, va, pb); } while (0)
#define SAGE_BODY3(MASKED_)                                                                          \
  do {                                                                                               \
    const int nx1 = cur == NST - 1 ? 0 : cur + 1;                                                    \
    const int nxp = PD == 1 ? nx1 : (nx1 == NST - 1 ? 0 : nx1 + 1);      /* stage of block j + PD */  \
    wait_all();                                                                                      \
    __syncthreads();                                                                                 \
    if (j + PD < nblk) issue(j + PD, nxp);                                                           \
    read_k(cur);                                                                                     \
    read_ds(cur, 0);                                                                                 \
    read_ds(cur, 1);                                                                                 \
    read_scales(cur);                                                                                \
    qk_tile<D, INT4>(ka, qreg, raw);                                                                 \
    Factors<GM> fn;                                                                                  \
    fn.set(dq, p.kappa, ks);                                                                         \
    SAGE_DEQ_ALL(MASKED_, j * BKV);                                                                  \
    alpha = update_max<D, INT4, GM, PVF>(st, sc, fn, m_sub);                                         \
    block_rescale<D>(st, alpha);                                                                     \
    v8i pb;                                                                                          \
    float ls = 0.0f;                                                                                 \
    SAGE_E3(0, MASKED_); SAGE_E3(1, MASKED_); SAGE_E3(2, MASKED_); SAGE_E3(3, MASKED_);              \
    read_v(cur);                                                                                     \
    SAGE_E3(4, MASKED_); SAGE_E3(5, MASKED_); SAGE_E3(6, MASKED_); SAGE_E3(7, MASKED_);              \
    st.l_run = __fmaf_rn(alpha, st.l_run, ls);                                                       \
    SAGE_P3(0); SAGE_P3(1); SAGE_P3(2); SAGE_P3(3); SAGE_P3(4); SAGE_P3(5); SAGE_P3(6); SAGE_P3(7);  \
    cur = nx1;                                                                                       \
  } while (0)
  int j = j_begin;
  // The workgroups of a CU do not advance alike: the SIMDs serve the oldest wavefront first (128 channels, three workgroups: 1.2 us a
  // block for the first, 2.5 for the last), so that the last of a launch end one after the other, each with more of its CU to itself than it can use.  Those that
  // start in the last round therefore begin at the highest priority and lower it as their keys run out: of workgroups that share
  // a CU the one with more left to do goes first, and they end together.  (Earlier rounds are better off uneven, their ends fall between the
  // others' blocks: 4096 tiles of 128 channels 572 -> 568 us, with every round 593.  Under a causal mask the tiles go out heaviest
  // first, and the oldest is the right one to be first: 8192 tokens, 64 channels 217 -> 222.)  Attention alone, us, without / with, 4096 keys, no mask:
  // 128 channels 512 tiles 94 / 87, 640 126 / 112, 768 132 / 121, 1024 173 / 164, 2048 328 / 316, 8-bit 768 141 / 133; 256 channels 512 138
  // / 132, 1024 266 / 261; 64 channels 1024 129 / 117, 4096 430 / 422; 256 tiles in three chunks of 88 blocks 167 / 156.
  constexpr bool EVEN_TAIL = !PACK && (!CAUSAL || SPLIT);
  constexpr unsigned SLOTS = 256 * attn_occupancy<D, GM, PVF>();
  if constexpr (OCC3) {
    if constexpr (EVEN_TAIL) {
      // (in stretches between the changes of priority; the loop itself knows nothing of them)
      int level = 0;
      if (blockIdx.x + SLOTS >= (unsigned)n_wg && n_wg > 256) {
        while (level < 3 && nblk - j <= tail_left<D>(level)) ++level;
        set_priority(3 - level);
      } else {
        level = 3;
      }
      for (;;) {
        const int stop = level < 3 ? min(n_plain, nblk - tail_left<D>(level)) : n_plain;
        for (; j < stop; ++j) SAGE_BODY3(false);
        if (j >= n_plain) break;
        set_priority(3 - ++level);
      }
    } else {
      for (; j < n_plain; ++j) SAGE_BODY3(false);
    }
    for (; j < n_act; ++j) SAGE_BODY3(true);
  } else {
    for (; j + 1 < n_plain; ++j) SAGE_BODY(false, false);
    if (j < n_plain) { SAGE_BODY(false, true); ++j; }      // the last unmasked block, a masked (or no) successor
    for (; j < n_act; ++j) SAGE_BODY(true, true);
  }
  // causal only: blocks past this wavefront's last query - keep up the copies and the barriers
  for (; j < nblk; ++j) {
    const int nx1 = cur == NST - 1 ? 0 : cur + 1;
    const int nxp = PD == 1 ? nx1 : (nx1 == NST - 1 ? 0 : nx1 + 1);
    wait_all();
    __syncthreads();
    if (j + PD < nblk) issue(j + PD, nxp);
    cur = nx1;
  }
#undef SAGE_BODY3
#undef SAGE_P3
#undef SAGE_E3
#undef SAGE_BODY
#undef SAGE_Y
#undef SAGE_X
#undef SAGE_DEQ_ALL
#undef SAGE_DEQ

  // ---- epilogue (Algorithm 1 last line): O / l / 448 * delta_V (+ mean(V) with the smooth-V
  // option, Sec. 3.4 last paragraph); l_run already carries the 448
  float l_tot = st.l_run;
  {
    const unsigned u = __float_as_uint(l_tot);
    const auto sw = __builtin_amdgcn_permlane32_swap(u, u, false, false);
    l_tot = __uint_as_float(sw[0]) + __uint_as_float(sw[1]);
  }
  if constexpr (SPLIT) {
    // a chunk of the keys: the sums stay under the chunk's own exponent offset and go to the merge kernel as they are
    const size_t prow = (size_t)((PACK ? tile : bh * p.nQb + qb) * p.splits + split) * BQ + w * WQ + n;
    if (PACK ? col_ok : query < sq.n) {
      if (half == 0) { p.part_el[prow * 2] = m_sub; p.part_el[prow * 2 + 1] = l_tot; }
#pragma unroll
      for (int ct = 0; ct < CT; ++ct) {
#pragma unroll
        for (int g = 0; g < 4; ++g) {
          const v4f o4 = {st.O[ct][4 * g], st.O[ct][4 * g + 1], st.O[ct][4 * g + 2], st.O[ct][4 * g + 3]};
          *reinterpret_cast<v4f*>(p.part_o + prow * D + 32 * ct + 8 * g + 4 * half) = o4;
        }
      }
    }
    return;
  }
  if (p.lse && half == 0 && query < sq.n) {
    // ln sum_t exp(sm_scale <q, k_t>) = ln 2 * (e + log2(l) + the row constant smoothing K dropped): l_tot is the
    // sum of 2^(S - e) under the final exponent offset e = m_sub, which survived the pipeline's last update
    // (that one saw a fully masked, stale block and left the running max where it was)
    p.lse[lse_index(p, sq, b, h, query)] =
        LN2 * ((m_sub + __builtin_amdgcn_logf(l_tot)) + lse_corr);
  }
  // One correctly rounded reciprocal per row instead of a division per element (64 of them were 4 % of
  // a tile of 64 blocks): O * fl32(1/l) is within one unit of the last FP32 place of fl32(O / l), far
  // below the rounding to the 16-bit output type that follows.
  const float inv_l = __fdiv_rn(1.0f, l_tot);
  if (query < sq.n) {
    unsigned short* orow = reinterpret_cast<unsigned short*>(p.out) +
                           row_offset(p.om, head_offset(p.om, (unsigned)bh), (int)sq.q0 + query);
#pragma unroll
    for (int ct = 0; ct < CT; ++ct) {
#pragma unroll
      for (int g = 0; g < 4; ++g) {
        const int c0 = 32 * ct + 8 * g + 4 * half;
        const v4f sc = *reinterpret_cast<const v4f*>(&s_vs[0][c0]);
        v4f vm = {0.0f, 0.0f, 0.0f, 0.0f};
        if (p.v_mean) vm = *reinterpret_cast<const v4f*>(&s_vs[1][c0]);
        float o4[4];
#pragma unroll
        for (int r = 0; r < 4; ++r) {
          o4[r] = __fmul_rn(__fmul_rn(st.O[ct][4 * g + r], inv_l), sc[r]);
          if (p.v_mean) o4[r] = __fadd_rn(o4[r], vm[r]);
        }
        *reinterpret_cast<uint2*>(orow + c0) = make_uint2(pack16x2<BF16>(o4[0], o4[1]), pack16x2<BF16>(o4[2], o4[3]));
      }
    }
  }
}

// Merge of the partial results of a tile's key chunks (Eq. 1 applied to disjoint key sets): under the largest of
// the chunks' exponent offsets e* the sums add up with weights 2^(e_s - e*); then the epilogue of Algorithm 1.
// A thread owns four channels of a row, d / 4 threads a row, and a workgroup takes 1024 / d of its tile's rows (grid: tiles,
// pieces of 1024 / d rows) - so a tile with few valid rows (a decode step) still spreads over a whole row of threads, and a
// row's chunks are read as contiguous 4 d bytes.
// PACK: the tiles of k_attn_fwd's packed form - row r of a tile is query r % n of head r / n of the KV head's group
// (n: the sequence's query count).
template <int D, bool BF16, bool PACK, int NB>
__global__ void __launch_bounds__(256) k_merge_splits(const AttnParams p) {
  constexpr int TPR = D / 4, RP = 256 / TPR;      // threads per row, rows per pass
  const int tile = blockIdx.x;
  const int t = threadIdx.x, c_lo = 4 * (t % TPR);
  for (int r = blockIdx.y * RP + t / TPR; r < BQ; r += RP * gridDim.y) {
    int bh = tile / p.nQb, qb = tile % p.nQb, query = qb * BQ + r;
    if constexpr (PACK) bh = (tile / p.Hkv) * p.H + (tile % p.Hkv) * (p.H / p.Hkv);      // the group's first head
    const Seq sq = seq_of(p.seq, (unsigned)(bh / p.H), p.N, p.Nk);
    if constexpr (PACK) {
      if (sq.n <= 0 || r >= (p.H / p.Hkv) * sq.n) return;
      bh += r / sq.n;
      qb = 0;
      query = r % sq.n;
    }
    const int b = bh / p.H, h = bh % p.H;
    const size_t bhkv = (size_t)b * p.Hkv + h / (p.H / p.Hkv);
    if (sq.nk == 0 || query >= sq.n) return;     // (rows ascend; a sequence without keys was written by the attention kernel)
    const size_t row0 = (size_t)tile * p.splits * BQ + r;       // this row in chunk 0; chunk s is s * BQ rows further
    // NB chunks at a time, all their loads issued before the first use (one round trip per batch, not one per chunk), those of
    // the first batch and delta_V together with the first look at the offsets that weight them all: bound by these trips, not by
    // bytes (512 queries on 16384 keys in three chunks 13.6 -> 12.8 us, a query of 128 heads in 16 chunks 7.0 -> 5.4).  The
    // chunks are summed in order
    float e[NB], lc[NB];
    v4f o4[NB];
    auto request = [&](int s0) {
#pragma unroll
      for (int i = 0; i < NB; ++i) {
        const size_t row = row0 + (size_t)min(s0 + i, p.splits - 1) * BQ;
        e[i] = p.part_el[row * 2];
        lc[i] = p.part_el[row * 2 + 1];
        o4[i] = *reinterpret_cast<const v4f*>(p.part_o + row * D + c_lo);
      }
    };
    request(0);
    const v4f vs = *reinterpret_cast<const v4f*>(p.v_scale + bhkv * D + c_lo);
    float e_max = -INFINITY;
    for (int s0 = NB; s0 < p.splits; s0 += NB) {
      float x[NB];
#pragma unroll
      for (int i = 0; i < NB; ++i) x[i] = p.part_el[(row0 + (size_t)min(s0 + i, p.splits - 1) * BQ) * 2];
#pragma unroll
      for (int i = 0; i < NB; ++i) e_max = fmaxf(e_max, x[i]);
    }
#pragma unroll
    for (int i = 0; i < NB; ++i) e_max = fmaxf(e_max, e[i]);
    float l = 0.0f;
    v4f acc = {0.0f, 0.0f, 0.0f, 0.0f};
    for (int s0 = 0;;) {
#pragma unroll
      for (int i = 0; i < NB; ++i) {
        if (s0 + i >= p.splits || e[i] == -INFINITY) continue;     // (an empty chunk left its sums unwritten)
        const float wgt = __builtin_amdgcn_exp2f(e[i] - e_max);
        l = __fmaf_rn(wgt, lc[i], l);
#pragma unroll
        for (int k = 0; k < 4; ++k) acc[k] = __fmaf_rn(wgt, o4[i][k], acc[k]);
      }
      s0 += NB;
      if (s0 >= p.splits) break;
      request(s0);
    }
    if (p.lse && c_lo == 0)
      p.lse[lse_index(p, sq, b, h, query)] =
          LN2 * ((e_max + __builtin_amdgcn_logf(l)) + p.q_corr[((size_t)bh * p.nQb + qb) * BQ + (query - qb * BQ)]);
    const float inv_l = __fdiv_rn(1.0f, l);
    unsigned short* orow = reinterpret_cast<unsigned short*>(p.out) +
                           row_offset(p.om, head_offset(p.om, (unsigned)bh), (int)sq.q0 + query) + c_lo;
    float y[4];
#pragma unroll
    for (int k = 0; k < 4; ++k) y[k] = __fmul_rn(__fmul_rn(acc[k], inv_l), vs[k]);
    if (p.v_mean) {
      const v4f vm = *reinterpret_cast<const v4f*>(p.v_mean + bhkv * D + c_lo);
#pragma unroll
      for (int k = 0; k < 4; ++k) y[k] = __fadd_rn(y[k], vm[k]);
    }
    *reinterpret_cast<uint2*>(orow) = make_uint2(pack16x2<BF16>(y[0], y[1]), pack16x2<BF16>(y[2], y[3]));
  }
}

// Integer score accumulators of one (128-query tile, 64-key block) through qk_tile.
template <int D, bool INT4>
__global__ void __launch_bounds__(256) k_debug_qk(const int8_t* __restrict__ q_codes,
                                                  const int8_t* __restrict__ k_codes, int q_tile,
                                                  int kv_block, int32_t* __restrict__ out) {
  constexpr int KCK = (int)(k_block_bytes(D, INT4) / 16);
  constexpr int NP = qk_pieces<D, INT4>();
  __shared__ v4i lds[KCK];
  const int t = threadIdx.x, lane = t & 63, w = t >> 6, n = lane & 31, half = lane >> 5;
  const v4i* gk = reinterpret_cast<const v4i*>(k_codes) + (size_t)kv_block * KCK;
  for (int i = t; i < KCK; i += 256) lds[i] = gk[i];
  __syncthreads();
  typename QkOperand<INT4>::type qreg[NP], ka[2 * NP];
  const v4i* gq = reinterpret_cast<const v4i*>(q_codes + (size_t)q_tile * q_slab_bytes(D, INT4)) +
                  (size_t)w * (q_slab_bytes(D, INT4) / 16 / (BQ / WQ));
#pragma unroll
  for (int s = 0; s < NP; ++s) qreg[s] = load_qk_operand<INT4>(gq, s, lane);
  // the block's operands come out of LDS through the attention kernel's own fetch code
  read_k_block<D, INT4>(&lds[0], lane, ka);
  v16i acc[2];
  qk_tile<D, INT4>(ka, qreg, acc);
#pragma unroll
  for (int kt = 0; kt < 2; ++kt) {
#pragma unroll
    for (int v = 0; v < 16; ++v)
      out[(w * WQ + n) * BKV + 32 * kt + 16 * half + v] = INT4 ? (int)__int_as_float(acc[kt][v]) : acc[kt][v];
  }
}

// One P~V-type MFMA on caller-provided operands (hardware check of the accumulation path).
__global__ void __launch_bounds__(64) k_debug_mfma_fp8(const v8i* __restrict__ a, const v8i* __restrict__ b,
                                                       const v16f* __restrict__ c, v16f* __restrict__ d) {
  const int l = threadIdx.x;
  d[l] = __builtin_amdgcn_mfma_scale_f32_32x32x64_f8f6f4(a[l], b[l], c[l], 0, 0, 0, 0, 0, 0);
}

hipError_t launch_debug_mfma_fp8(const void* a, const void* b, const float* c, float* d, hipStream_t s) {
  k_debug_mfma_fp8<<<1, 64, 0, s>>>((const v8i*)a, (const v8i*)b, (const v16f*)c, (v16f*)d);
  return hipGetLastError();
}

template <int D> constexpr int MERGE_ROWS = 1024 / D;      // rows a workgroup of k_merge_splits takes

// Batches of four where there are no more chunks (of eight, the places past the last are loads all the same: 512 queries on 16384 keys in
// three chunks, whole call 246.9 -> 243.6 us).
template <int D, bool PACK>
static hipError_t launch_merge_t(const Dims& Dm, const AttnParams& p, dim3 grid, hipStream_t s) {
  const bool four = Dm.splits <= 4;
  if (Dm.bf16) { if (four) k_merge_splits<D, true, PACK, 4><<<grid, 256, 0, s>>>(p); else k_merge_splits<D, true, PACK, 8><<<grid, 256, 0, s>>>(p); }
  else         { if (four) k_merge_splits<D, false, PACK, 4><<<grid, 256, 0, s>>>(p); else k_merge_splits<D, false, PACK, 8><<<grid, 256, 0, s>>>(p); }
  return hipGetLastError();
}
template <int D>
static hipError_t launch_merge_packed_t(const Dims& Dm, const AttnParams& p, hipStream_t s) {
  const int rows = min(BQ, Dm.H / Dm.Hkv * Dm.N);
  const dim3 grid(p.total_tiles, (rows + MERGE_ROWS<D> - 1) / MERGE_ROWS<D>);
  return launch_merge_t<D, true>(Dm, p, grid, s);
}
hipError_t launch_merge_packed(const Dims& Dm, const AttnParams& p, hipStream_t s) {
  return Dm.d == 256 ? launch_merge_packed_t<256>(Dm, p, s)
       : Dm.d == 128 ? launch_merge_packed_t<128>(Dm, p, s) : launch_merge_packed_t<64>(Dm, p, s);
}

template <int D, bool INT4, bool CAUSAL, bool BF16, int GM, int PVF>
static hipError_t launch_attention_g(const Dims& Dm, const Ptrs& P, hipStream_t s) {
  AttnParams p = attn_params(Dm, P);
  if constexpr (GM == 0 && PVF == PV_E4M3) {        // (the key split comes with the default groups and data type)
    if (Dm.pack) {                                  // packed tiles: one per (batch, KV head), any number of chunks
      p.total_tiles = Dm.B * Dm.Hkv;
      const int grid = 8 * ((p.total_tiles * Dm.splits + 7) / 8);
      k_attn_fwd<D, INT4, CAUSAL, BF16, GM, PVF, true, true><<<grid, 256, 0, s>>>(p);
      return launch_merge_packed(Dm, p, s);
    }
    if (Dm.splits > 1) {
      const int grid = 8 * ((p.total_tiles * Dm.splits + 7) / 8);
      k_attn_fwd<D, INT4, CAUSAL, BF16, GM, PVF, true><<<grid, 256, 0, s>>>(p);
      return launch_merge_t<D, false>(Dm, p, dim3(p.total_tiles, BQ / MERGE_ROWS<D>), s);
    }
  }
  const int grid = 8 * ((p.total_tiles + 7) / 8);
  k_attn_fwd<D, INT4, CAUSAL, BF16, GM, PVF><<<grid, 256, 0, s>>>(p);
  return hipGetLastError();
}
template <int D, bool INT4, bool CAUSAL, bool BF16>
static hipError_t launch_attention_t(const Dims& Dm, const Ptrs& P, hipStream_t s) {
  // the other data types of P~V come with the default key groups only
  if (Dm.pvf == PV_E5M2) return launch_attention_g<D, INT4, CAUSAL, BF16, 0, PV_E5M2>(Dm, P, s);
  if (Dm.pvf == PV_INT8) return launch_attention_g<D, INT4, CAUSAL, BF16, 0, PV_INT8>(Dm, P, s);
  if (Dm.kg == KGROUP) return launch_attention_g<D, INT4, CAUSAL, BF16, 0, PV_E4M3>(Dm, P, s);
  if (Dm.kg == 4) return launch_attention_g<D, INT4, CAUSAL, BF16, 1, PV_E4M3>(Dm, P, s);
  return launch_attention_g<D, INT4, CAUSAL, BF16, 2, PV_E4M3>(Dm, P, s);
}

hipError_t launch_attention(const Dims& D, const Ptrs& P, hipStream_t s) {
#define SAGE_ATT(DD, I4, CA, BF) return launch_attention_t<DD, I4, CA, BF>(D, P, s)
#define SAGE_ATT_BF(DD, I4, CA) do { if (D.bf16) SAGE_ATT(DD, I4, CA, true); else SAGE_ATT(DD, I4, CA, false); } while (0)
#define SAGE_ATT_CA(DD, I4) do { if (D.causal) SAGE_ATT_BF(DD, I4, true); else SAGE_ATT_BF(DD, I4, false); } while (0)
  if (D.d == 256)      { if (D.int4) SAGE_ATT_CA(256, true); else SAGE_ATT_CA(256, false); }
  else if (D.d == 128) { if (D.int4) SAGE_ATT_CA(128, true); else SAGE_ATT_CA(128, false); }
  else                 { if (D.int4) SAGE_ATT_CA(64, true); else SAGE_ATT_CA(64, false); }
#undef SAGE_ATT_CA
#undef SAGE_ATT_BF
#undef SAGE_ATT
}

hipError_t launch_debug_qk(const Dims& D, const Ptrs& P, int b, int h, int q_tile, int kv_block,
                           int32_t* out, hipStream_t s) {
  const size_t bh = (size_t)b * D.H + h;
  const size_t bhkv = (size_t)b * D.Hkv + h / (D.H / D.Hkv);
  const int8_t* qc = P.q_codes + bh * (size_t)D.nQb * q_slab_bytes(D.d, D.int4);
  const int8_t* kc = P.k_codes + bhkv * (size_t)D.nKb * k_block_bytes(D.d, D.int4);
  if (D.d == 256) {
    if (D.int4) k_debug_qk<256, true><<<1, 256, 0, s>>>(qc, kc, q_tile, kv_block, out);
    else k_debug_qk<256, false><<<1, 256, 0, s>>>(qc, kc, q_tile, kv_block, out);
  } else if (D.d == 128) {
    if (D.int4) k_debug_qk<128, true><<<1, 256, 0, s>>>(qc, kc, q_tile, kv_block, out);
    else k_debug_qk<128, false><<<1, 256, 0, s>>>(qc, kc, q_tile, kv_block, out);
  } else {
    if (D.int4) k_debug_qk<64, true><<<1, 256, 0, s>>>(qc, kc, q_tile, kv_block, out);
    else k_debug_qk<64, false><<<1, 256, 0, s>>>(qc, kc, q_tile, kv_block, out);
  }
  return hipGetLastError();
}

}  // namespace sage
