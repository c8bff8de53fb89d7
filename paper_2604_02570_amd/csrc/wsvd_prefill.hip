// Causal attention of a block of query tokens over the int8 latent cache, tiled for the matrix cores (the attention
// of prefilling, Section 3.4, in latent space).
//
// With no rotation between the reconstruction and the product, q K^T = (q B_K^T) C_K^T and P V = (P C_V) B_V: the
// whole score / softmax / value loop runs on latents of dimension r instead of keys and values of dimension d.
//   prologue  Q~^T [r x 32 queries] = B_K q^T                       bf16 MFMA, operands straight from global memory
//   loop      S^T [32 keys x 32 queries] = C_K Q~^T                 fp16 MFMA: codes are exact in fp16, Q~ is an fp16 pair
//             online softmax down the columns (a lane owns one query column)
//             U^T [r x 32 queries] += (diag(s_V) C_V)^T P           fp16 MFMA: code * scale and P rounded to fp16 (2^-12
//                                                                   relative each)
//   epilogue  O^T [d x 32 queries] = B_V^T (U / l)                  bf16 MFMA, U an bf16 pair
//
// The loop is bound by the vector ALU (81 vector instructions per 32 x 32 block and wave, of which the 16 exponentials run
// at half rate, 8.3 against 4.2 cycles: a third of it; the products hide behind it only in part, about 10 cycles each
// remain), so it is laid out to spend few vector instructions per score:
//   * the QW waves of a key group convert the codes of QW cache blocks to fp16 operands once, one block each, through two
//     LDS stages, and each attends its own 32 query rows to all of them (48 of the conversion's instructions per block
//     become 12 and 6 LDS reads; a single wave of rows converts for itself, without LDS: 64 x 9 tokens of rank 64 over 1000
//     keys 67 -> 60 us);
//   * the key rows of the score product are taken in the order 16 g + 4 m + j for accumulator register 4 m + j of lane
//     half g (the lane of the A operand loads that token's codes).  The weights a lane ends up with are then, in register
//     order, the operand the value product wants: P never leaves the registers, and the 16 scales a lane needs, of K as
//     of V, are 16 consecutive fp16 values of the metadata plane;
//   * score * scale - reference is one mixed-precision multiply-add.  The reference of the exponentials is the running
//     maximum, so that the largest weight of a column is exactly 1 in fp16; a block whose scores stay below it (told by
//     the sign of the largest difference) leaves the accumulators alone and exchanges nothing between lane halves (the
//     masked and the plain form of the loop stay apart: one loop with both copied all accumulators per block, 0.47 ms);
//   * the weights are summed in fp32, before they are rounded to fp16 for the value product.
// 16 x 2048 tokens, 32 heads, r = 32: 0.43 ms (0.53 ms with one wave per 32 rows converting for itself, the maximum
// exchanged every block and P through LDS).  A reference that is moved only when a block's weights sum to more than 64,
// with the weights summed as the fp16 values: the same time there, but the largest weight is then not exact (error against
// 64 bits up to 2.14e-4 where this has 2.12e-4, and 2.5e-4 with the sum in fp32).  With scores so small that such a
// reference never moves, the maxima that do cost 7 % (0.53 ms against 0.49 at the clock that data leaves, 0.64 with one wave
// per 32 rows).  Tried and slower: two query
// blocks per wave without LDS (193 registers, two waves per SIMD; three waves spill), the next block's score products issued
// under the softmax.
//
// A workgroup is QW x KG waves: KG key groups take every KG-th stage of QW blocks, their (m, l, U) meet in LDS.  A query
// row is a (token, head) pair, token-major, so the G heads that share a kv head share the stream too.  The cache blocks
// are read in the layout the decode kernels use (a 32-token block of the K plane is a ready-made operand with row = token,
// one of the V plane with row = dim).
// 32x32 accumulator layout throughout: lane L holds column L % 32, rows 8 (v / 4) + 4 (L / 32) + v % 4, v = 0..15.
#include <algorithm>
#include <type_traits>
#include "wsvd_dev.h"
#include "wsvd_internal.h"

namespace {

struct PrefillParams {
  const uint16_t* q;          // bf16 [B, Hkv, NR, d], NR = nq * G query rows per kv head (row = token * G + head)
  const uint16_t* BK;         // bf16 [Hkv, R, d]
  const uint16_t* BV;
  const uint8_t* k_codes;
  const uint8_t* v_codes;
  const uint16_t* k_meta;
  const uint16_t* v_meta;
  const int* seq_lens;
  float* out;                 // fp32 [B, Hkv, NR, d]
  int B, Hkv, G, d, t_cap, nq, n_after, NR;
  float c_scale;              // sm_scale * log2(e)
  // paged cache only (else null): the planes are pools of n_pages pages, a page = page_rows rows of every kv head in the
  // layout of a contiguous plane; block_table [B][max_pages]
  const int* block_table;
  int page_rows, max_pages, n_pages;
};

// x as an fp16 pair hi + lo; the fp32 value is pinned in a register so that hi is formed once (a fused
// multiply-convert would otherwise round it a second way for the subtraction)
WSVD_DEV void split_f16(float x, _Float16& hi, _Float16& lo) {
  asm volatile("" : "+v"(x));
  hi = (_Float16)x;
  lo = (_Float16)(x - (float)hi);
}
// x as a bf16 pair (truncation: hi + lo reproduces x to 2^-16 relative)
WSVD_DEV void split_bf16(float x, uint32_t& hi, uint32_t& lo) {
  hi = __float_as_uint(x) & 0xFFFF0000u;
  lo = __float_as_uint(x - __uint_as_float(hi)) & 0xFFFF0000u;
}

// a block's operands: from the stage that the waves of a key group share, or converted by the wave for itself
template <int KK>
struct StageOperands {
  const uint8_t* src;
  int lane, g2;
  WSVD_DEV v8f16 k(int s) const { return *(const v8f16*)(src + s * 1024 + lane * 16); }
  WSVD_DEV v8f16 ks(int s) const { return *(const v8f16*)(src + 4 * KK * 1024 + 32 * g2 + 16 * s); }
  WSVD_DEV v8f16 v(int kk, int s) const { return *(const v8f16*)(src + (2 * KK + 2 * kk + s) * 1024 + lane * 16); }
};
template <int KK>
struct OwnOperands {
  v8f16 kc[2 * KK], vc[KK][2], sc[2];
  WSVD_DEV v8f16 k(int s) const { return kc[s]; }
  WSVD_DEV v8f16 ks(int s) const { return sc[s]; }
  WSVD_DEV v8f16 v(int kk, int s) const { return vc[kk][s]; }
};

enum { kFirst, kWhole, kPart, kAny };      // what a wave's queries see of a key block, see there

// (Rank 64 in key groups: two waves per SIMD even where the registers would hold three.  The waves of such a launch are few and of
// unequal length; with three a CU takes more of the long ones than its neighbour: 5 x 1007 tokens, 8 heads, 39.6 us, with two 36.2.)
template <int R, int D, int QW, int KG>
__global__ __launch_bounds__(64 * QW * KG) __attribute__((amdgpu_waves_per_eu(R == 32 ? 4 : 2, R == 64 && KG > 1 ? 2 : 8)))
void k_prefill_attn(PrefillParams p) {
  constexpr int KK = R / 32;
  constexpr bool OWN = QW == 1;
  constexpr int BLK = 4 * KK * 1024 + 64;                               // one cache block as operands: K, V', K scales
  constexpr int STAGE = QW * BLK;                                       // QW blocks: one converted by each wave of a group
  constexpr int STAGES = !OWN ? KG * 2 * STAGE : 16, MERGE = KG > 1 ? QW * KG * (KK * 4096 + 256) : 0;
  __shared__ __attribute__((aligned(16))) uint8_t lds[STAGES > MERGE ? STAGES : MERGE];

  const int lane = threadIdx.x & 63, n = lane & 31, g2 = lane >> 5;
  const int wave = __builtin_amdgcn_readfirstlane(threadIdx.x >> 6);    // (uniform: block addresses stay scalar)
  const int qw = wave % QW, kg = wave / QW;
  // the last query blocks see the most keys: they are started first, so that the launch does not end on its longest waves
  const int kv = blockIdx.x, qb = (gridDim.y - 1 - blockIdx.y) * QW + qw, b = blockIdx.z;
  const size_t ph = (size_t)b * p.Hkv + kv;
  const int perm = 16 * ((n >> 2) & 1) + 4 * (n >> 3) + (n & 3);
  const int rho_c = min(qb * 32 + n, p.NR - 1);                         // this lane's query row
  // nothing here depends on the length: queries, B_K and the length itself travel in one round trip
  v8bf16 bq[D / 16], bk[KK][D / 16];
#pragma unroll
  for (int ks = 0; ks < D / 16; ks++) bq[ks] = *(const v8bf16*)(p.q + (ph * p.NR + rho_c) * D + 8 * g2 + 16 * ks);
#pragma unroll
  for (int kk = 0; kk < KK; kk++)
#pragma unroll
    for (int ks = 0; ks < D / 16; ks++) bk[kk][ks] = *(const v8bf16*)(p.BK + ((size_t)kv * R + 32 * kk + perm) * D + 16 * ks + 8 * g2);
  const int n_eff = min(max(p.seq_lens[b] - p.n_after, 0), p.t_cap);
  const int lim = n_eff - p.nq + rho_c / p.G + 1;                       // this query sees keys [0, lim); may be <= 0
  // rows are token-major: a wave's last row sees most of its keys, the workgroup's last row most of all.
  // (readfirstlane: the divisions run on the vector ALU, the values are uniform)
  auto sees = [&](int row) { return __builtin_amdgcn_readfirstlane(n_eff - p.nq + min(row, p.NR - 1) / p.G + 1); };
  const int lim_wg = sees((qb - qw) * 32 + 32 * QW - 1);
  const int n_kblocks = lim_wg > 0 ? (lim_wg + 31) >> 5 : 0;            // of the workgroup
  if (n_kblocks == 0) {                                                 // nothing visible to any row of the workgroup
    int lane_z = lane_number();                                         // (of its own: no register is held through the loop for it)
    asm volatile("" : "+v"(lane_z));
    const int row = qb * 32 + (lane_z & 31), gz = lane_z >> 5;
    float* const orow = p.out + (ph * p.NR + min(row, p.NR - 1)) * D;
    if (row < p.NR && kg == 0)
      for (int c = gz * (D / 2); c < (gz + 1) * (D / 2); c++) orow[c] = 0.f;
    return;
  }
  const int lim_max = qb * 32 < p.NR ? sees(qb * 32 + 31) : 0, lim_min = sees(qb * 32);
  const int kb_end = lim_max > 0 ? (lim_max + 31) >> 5 : 0;             // blocks this wave's rows see any key of
  const int kb_full = lim_min > 0 ? min(lim_min >> 5, kb_end) : 0;      // blocks every row of the wave sees whole: no masks

  // ---- Q~^T = B_K q^T.  Row i of the A operand carries latent dim pi(i) = 16 ((i >> 2) & 1) + 4 (i >> 3) + (i & 3) of
  // its 32-dim block, so that accumulator register v of lane half g2 is dim 16 g2 + v: the order the K blocks use.
  v8f16 qh[2 * KK], ql[2 * KK];                                         // 16-dim steps of the score contraction
#pragma unroll
  for (int kk = 0; kk < KK; kk++) {
    v16f qt;
#pragma unroll
    for (int v = 0; v < 16; v++) qt[v] = 0.f;
#pragma unroll
    for (int ks = 0; ks < D / 16; ks++) qt = mfma_bf16(bk[kk][ks], bq[ks], qt);
#pragma unroll
    for (int v = 0; v < 16; v++) {
      _Float16 h, l;
      split_f16(qt[v] * p.c_scale, h, l);
      qh[2 * kk + (v >> 3)][v & 7] = h;
      ql[2 * kk + (v >> 3)][v & 7] = l;
    }
  }

  const uint8_t* kplane = p.k_codes + ph * (size_t)p.t_cap * R;
  const uint8_t* vplane = p.v_codes + ph * (size_t)p.t_cap * R;
  const uint16_t* kmeta = p.k_meta + ph * (size_t)p.t_cap;
  const uint16_t* vmeta = p.v_meta + ph * (size_t)p.t_cap;

  float m_ref = -INFINITY, l_run = 0.f;                                 // l_run: this lane's share of its column's sum
  v16f U[KK];
#pragma unroll
  for (int kk = 0; kk < KK; kk++)
#pragma unroll
    for (int v = 0; v < 16; v++) U[kk][v] = 0.f;

  // the raw block this wave converts next, requested one stage ahead: codes of both planes, K scales (lanes 0..3 hold the
  // 32 tokens'), V scales of the lane half's 16 tokens
  v4i kc[KK], vc[KK], ks16[OWN ? 2 : 1], vs16[2];
  // paged cache: the table entries of the first 64 pages, one per lane, fetched once; a block's page is then a lane
  // read with a wave-uniform index (a 32-token block never straddles pages).  Entries outside the pools read page 0
  // (blocks past a sequence's end are never consumed; a bad entry under live rows is the append's to report).
  int page_entry = 0;
  if (p.block_table) page_entry = p.block_table[(size_t)b * p.max_pages + min(lane, p.max_pages - 1)];
  const uint32_t k_lane = (g2 * 32 + perm) * 16, v_lane = lane * 16;    // byte offsets (32-bit: scalar base + lane offset)
  auto load_block = [&](int kb) {
    const uint8_t *kp = kplane, *vp = vplane;
    const uint16_t *km = kmeta, *vm = vmeta;
    if (p.block_table) {
      const int bpp = p.page_rows >> 5;                                 // blocks per page
      const int pg = __builtin_amdgcn_readfirstlane(min(kb / bpp, p.max_pages - 1));
      int e = pg < 64 ? __builtin_amdgcn_readlane(page_entry, pg) : p.block_table[(size_t)b * p.max_pages + pg];
      e = (e >= 0 && e < p.n_pages) ? e : 0;
      const size_t slot = (size_t)e * p.Hkv + kv;
      kp = p.k_codes + slot * (size_t)p.page_rows * R; vp = p.v_codes + slot * (size_t)p.page_rows * R;
      km = p.k_meta + slot * (size_t)p.page_rows; vm = p.v_meta + slot * (size_t)p.page_rows;
      kb -= pg * bpp;
    }
    const size_t off = (size_t)kb * (32 * R);
#pragma unroll
    for (int kk = 0; kk < KK; kk++) {
      kc[kk] = *(const v4i*)((kp + off + kk * 1024) + k_lane);          // (plain loads: the other query blocks of this
      vc[kk] = *(const v4i*)((vp + off + kk * 1024) + v_lane);          //  sequence and head read the same blocks again)
    }
    if (!OWN) ks16[0] = *(const v4i*)(km + kb * 32 + 8 * (lane & 3));
#pragma unroll
    for (int s = 0; s < 2; s++) {
      if constexpr (OWN) ks16[s] = *(const v4i*)(km + kb * 32 + 16 * g2 + 8 * s);
      vs16[s] = *(const v4i*)(vm + kb * 32 + 16 * g2 + 8 * s);
    }
  };
  // ... as operands.  V' = code * s_V in fp16 (the token scales are fp16 already: one packed multiply per two elements);
  // tokens no query of the workgroup sees (among them rows never written, whose scale may be anything) contribute 0.
  auto value_scales = [&](v8f16 (&sv8)[2], int kb) {
    sv8[0] = __builtin_bit_cast(v8f16, vs16[0]); sv8[1] = __builtin_bit_cast(v8f16, vs16[1]);
    if (kb * 32 + 32 > lim_wg) {
#pragma unroll
      for (int s = 0; s < 2; s++)
#pragma unroll
        for (int e = 0; e < 8; e++)
          if (kb * 32 + 16 * g2 + 8 * s + e >= lim_wg) sv8[s][e] = (_Float16)0;
    }
  };
  auto convert_block = [&](uint8_t* dst, int kb) {                      // into the wave's slot of a stage
    v8f16 sv8[2];
    value_scales(sv8, kb);
#pragma unroll
    for (int kk = 0; kk < KK; kk++)
#pragma unroll
      for (int h = 0; h < 2; h++) {
        *(v8f16*)(dst + (2 * kk + h) * 1024 + lane * 16) = codes_f16(kc[kk][2 * h], kc[kk][2 * h + 1]);
        *(v8f16*)(dst + (2 * KK + 2 * kk + h) * 1024 + lane * 16) = codes_f16(vc[kk][2 * h], vc[kk][2 * h + 1]) * sv8[h];
      }
    if (lane < 4) *(v4i*)(dst + 4 * KK * 1024 + lane * 16) = ks16[0];
  };
  auto own_operands = [&](OwnOperands<KK>& o, int kb) {                 // (nobody to share them with)
    v8f16 sv8[2];
    value_scales(sv8, kb);
#pragma unroll
    for (int kk = 0; kk < KK; kk++)
#pragma unroll
      for (int h = 0; h < 2; h++) {
        o.kc[2 * kk + h] = codes_f16(kc[kk][2 * h], kc[kk][2 * h + 1]);
        o.vc[kk][h] = codes_f16(vc[kk][2 * h], vc[kk][2 * h + 1]) * sv8[h];
      }
    o.sc[0] = __builtin_bit_cast(v8f16, ks16[0]); o.sc[1] = __builtin_bit_cast(v8f16, ks16[OWN ? 1 : 0]);
  };

  // over a column's rows, half of which the other half of the wave holds (through LDS where a register is left for the index: the
  // exchange of halves takes two at once)
  auto column_max = [&](float x) { return OWN ? fmaxf(x, __shfl_xor(x, 32)) : halves_max(x); };
  // op: the block's operands, each asked for where it is used (k(s), scales ks(s), v(kk, s))
  // kFirst: nothing seen yet, every query sees the whole block; kWhole: every query does; kPart: every query has a reference,
  // some see a part; kAny: everything else.  (68, 68, 100 and 200 vector instructions; with the general form for the first and the
  // last block of every prompt, and the output's operands from single elements of B_V: 4 x 100 tokens of rank 64 9.3 -> 8.4 us,
  // 16 x 32 over 232 keys 11.2 -> 10.9, 2 x 700 21.2 -> 20.9, 16 x 2048 418 -> 416.)
  auto block = [&](const auto& op, int kb, auto form_c) {
    constexpr int FORM = decltype(form_c)::value;
    // scores: rows = the block's 32 tokens (register v of half g2 = token 16 g2 + v), columns = the 32 queries
    const v16f zero16 = {0.f, 0.f, 0.f, 0.f, 0.f, 0.f, 0.f, 0.f, 0.f, 0.f, 0.f, 0.f, 0.f, 0.f, 0.f, 0.f};
    v16f S;
#pragma unroll
    for (int s = 0; s < 2 * KK; s++) {
      const v8f16 aK = op.k(s);
      S = mfma_f16(aK, qh[s], s ? S : zero16);                          // (a constant-zero addend: no registers to clear)
      S = mfma_f16(aK, ql[s], S);
    }
    const v8f16 sk8[2] = {op.ks(0), op.ks(1)};
    v8f16 aV[KK][2];
#pragma unroll
    for (int kk = 0; kk < KK; kk++)
#pragma unroll
      for (int s = 0; s < 2; s++) aV[kk][s] = op.v(kk, s);
    float x[16];
    if constexpr (FORM == kFirst) {
      float bmax = -INFINITY;
#pragma unroll
      for (int v = 0; v < 16; v++) {
        x[v] = S[v] * (float)sk8[v >> 3][v & 7];
        bmax = fmaxf(bmax, x[v]);
      }
      m_ref = column_max(bmax);
      const float m_fin = fmaxf(m_ref, -3.402823466e38f);               // (every score -inf: no reference yet, weights 0)
#pragma unroll
      for (int v = 0; v < 16; v++) x[v] -= m_fin;
    } else if constexpr (FORM == kAny) {
      float bmax = -INFINITY;
#pragma unroll
      for (int v = 0; v < 16; v++) {
        const float sc = S[v] * (float)sk8[v >> 3][v & 7];
        x[v] = kb * 32 + 16 * g2 + v < lim ? sc : -INFINITY;
        bmax = fmaxf(bmax, x[v]);
      }
      bmax = column_max(bmax);                                          // the other half holds the column's other rows
      const float m_new = fmaxf(m_ref, bmax);
      const float alpha = m_ref == -INFINITY ? 0.f : __builtin_amdgcn_exp2f(m_ref - m_new);
#pragma unroll
      for (int v = 0; v < 16; v++) x[v] = x[v] == -INFINITY ? -INFINITY : x[v] - m_new;   // (no key seen yet: m_new = -inf)
      m_ref = m_new; l_run *= alpha;
#pragma unroll
      for (int kk = 0; kk < KK; kk++)
#pragma unroll
        for (int v = 0; v < 16; v++) U[kk][v] *= alpha;
    } else {
      float bmax = -INFINITY;
#pragma unroll
      for (int v = 0; v < 16; v++) {
        x[v] = fmaf(S[v], (float)sk8[v >> 3][v & 7], -m_ref);           // (m_ref is finite here)
        if constexpr (FORM == kPart) x[v] = v < lim - kb * 32 - 16 * g2 ? x[v] : -INFINITY;
        bmax = fmaxf(bmax, x[v]);
      }
      if (__builtin_amdgcn_ballot_w64(bmax > 0.f) != 0) {               // some column's maximum moves
        bmax = column_max(bmax);
        const float m_new = m_ref + fmaxf(bmax, 0.f), d = m_new - m_ref;
        const float alpha = __builtin_amdgcn_exp2f(-d);
        m_ref = m_new; l_run *= alpha;
#pragma unroll
        for (int v = 0; v < 16; v++) x[v] -= d;
#pragma unroll
        for (int kk = 0; kk < KK; kk++)
#pragma unroll
          for (int v = 0; v < 16; v++) U[kk][v] *= alpha;
      }
    }
    // weights: their sum in fp32, as operands of the value product in fp16.  Registers 8 s .. 8 s + 7 are tokens
    // 16 g2 + 8 s .. + 7, the operand of its step s.
    v8f16 bp[2];
    float psum = 0.f;
#pragma unroll
    for (int v = 0; v < 16; v++) {
      const float w = __builtin_amdgcn_exp2f(x[v]);
      psum += w;
      bp[v >> 3][v & 7] = (_Float16)w;
    }
    l_run += psum;
    // U^T += V'^T P: rows = latent dims, columns = queries
#pragma unroll
    for (int s = 0; s < 2; s++)
#pragma unroll
      for (int kk = 0; kk < KK; kk++) U[kk] = mfma_f16(aV[kk][s], bp[s], U[kk]);
  };

  // blocks kb, kb + STEP, .. below end in loops by their form: the first one (a column without a key yet has no reference), the
  // blocks seen whole, the last ones.  (One loop with a choice inside copies the accumulators of both forms in every block.)
  constexpr std::integral_constant<int, kFirst> first_c{};
  constexpr std::integral_constant<int, kWhole> whole_c{};
  constexpr std::integral_constant<int, kPart> part_c{};
  constexpr std::integral_constant<int, kAny> any_c{};
  auto no_reference = [&] { return __builtin_amdgcn_ballot_w64(m_ref == -INFINITY) != 0; };
  if constexpr (OWN) {
    // ---- one wave of rows per key group: its blocks go straight to registers, every KG-th one
    load_block(min(kg, n_kblocks - 1));
    auto next = [&](int kb, auto form_c) {
      OwnOperands<KK> o;
      own_operands(o, kb);
      load_block(min(kb + KG, n_kblocks - 1));                          // (after the last block: the last one again, unused)
      block(o, kb, form_c);
    };
    int kb = kg;
    bool open = kb >= kb_full;                                          // some column may have no reference yet
    if (!open) { next(kb, first_c); kb += KG; open = __builtin_expect(no_reference(), 0); }
    if (open)
      for (; kb < n_kblocks && no_reference(); kb += KG) next(kb, any_c);
    for (; kb < kb_full; kb += KG) next(kb, whole_c);
    for (; kb < n_kblocks; kb += KG) next(kb, part_c);
  } else {
    // ---- stages of QW blocks: every wave converts one block of the next stage, then all of them attend to the whole
    // current one; a key group takes every KG-th stage
    uint8_t* const stage = lds + kg * (2 * STAGE);
    const int n_stages = (n_kblocks + QW - 1) / QW, n_iter = (n_stages + KG - 1) / KG;
    auto own_block = [&](int it) { return (it * KG + kg) * QW + qw; };  // (may lie past the end: clamped loads, never read)
    load_block(min(own_block(0), n_kblocks - 1));
    convert_block(stage + qw * BLK, own_block(0));
    load_block(min(own_block(1), n_kblocks - 1));
    __syncthreads();
    for (int it = 0; it < n_iter; it++) {
      if (it + 1 < n_iter) {
        convert_block(stage + ((it + 1) & 1) * STAGE + qw * BLK, own_block(it + 1));
        load_block(min(own_block(it + 2), n_kblocks - 1));
      }
      const uint8_t* src = stage + (it & 1) * STAGE;
      const int kb0 = (it * KG + kg) * QW, j_full = min(kb_full - kb0, QW), j_end = min(kb_end - kb0, QW);
      auto staged = [&](int j, auto form_c) { block(StageOperands<KK>{src + j * BLK, lane, g2}, kb0 + j, form_c); };
      int j = 0;
      bool open = it != 0 || j_full <= 0;
      if (!open) { staged(j++, first_c); open = __builtin_expect(no_reference(), 0); }
      if (open)
        for (; j < j_end && no_reference(); j++) staged(j, any_c);
      for (; j < j_full; j++) staged(j, whole_c);
      for (; j < j_end; j++) staged(j, part_c);
      __syncthreads();
    }
  }

  float L = OWN ? l_run + __shfl_xor(l_run, 32) : halves_sum(l_run);
  if constexpr (KG > 1) {
    // the key groups' partial results: every group's wave of the same rows folds all of them in group order, then takes its
    // share of the output channels  (LDS: U in register order, then m and l per query; the last barrier has passed)
    float* const mine = (float*)(lds + (size_t)wave * (KK * 4096 + 256));
#pragma unroll
    for (int kk = 0; kk < KK; kk++)
#pragma unroll
      for (int v = 0; v < 16; v++) mine[(kk * 16 + v) * 64 + lane] = U[kk][v];
    if (g2 == 0) { mine[KK * 1024 + n] = m_ref; mine[KK * 1024 + 32 + n] = L; }
    __syncthreads();
    float m = -INFINITY;
    L = 0.f;
#pragma unroll
    for (int kk = 0; kk < KK; kk++)
#pragma unroll
      for (int v = 0; v < 16; v++) U[kk][v] = 0.f;
#pragma unroll
    for (int g = 0; g < KG; g++) m = fmaxf(m, ((const float*)(lds + (size_t)(g * QW + qw) * (KK * 4096 + 256)))[KK * 1024 + n]);
#pragma unroll
    for (int g = 0; g < KG; g++) {
      const float* part = (const float*)(lds + (size_t)(g * QW + qw) * (KK * 4096 + 256));
      const float mg = part[KK * 1024 + n];
      const float f = mg == -INFINITY ? 0.f : __builtin_amdgcn_exp2f(mg - m);     // (a group that saw no key: U = 0, l = 0)
      L = fmaf(f, part[KK * 1024 + 32 + n], L);
#pragma unroll
      for (int kk = 0; kk < KK; kk++)
#pragma unroll
        for (int v = 0; v < 16; v++) U[kk][v] = fmaf(f, part[(kk * 16 + v) * 64 + lane], U[kk][v]);
    }
  }

  // ---- O^T = B_V^T (U / l).  Register v of U[kk] in lane half g2 is latent dim 32 kk + 8 (v / 4) + 4 g2 + v % 4; the A
  // operand gathers the rows of B_V in that order (all of the wave's output channels in one round trip).
  // (the lane's number and row anew from the hardware: no register, and no scratch memory, holds them through the loop)
  int lane_e = lane_number();
  asm volatile("" : "+v"(lane_e));
  const int n_e = lane_e & 31, g_e = lane_e >> 5;
  // Where a wave has two blocks of 32 channels, they are the even and the odd ones of 64: a dword holds an element of either.
  constexpr int NRB = D / 32 / KG < 1 ? 1 : D / 32 / KG;                // blocks of 32 output channels per wave
  constexpr bool PAIRS = NRB % 2 == 0;
  v4i av[NRB][KK][2];
#pragma unroll
  for (int t = 0; t < NRB; t += PAIRS ? 2 : 1) {
    const int c = PAIRS ? 64 * (kg + t / 2 * KG) + 2 * n_e : 32 * min(kg + t * KG, D / 32 - 1) + n_e;     // (first) output channel of this lane's A row
#pragma unroll
    for (int kk = 0; kk < KK; kk++)
#pragma unroll
      for (int s = 0; s < 2; s++)
#pragma unroll
        for (int e = 0; e < 4; e++) {
          const int v0 = 8 * s + 2 * e, v1 = v0 + 1;
          const int j0 = 32 * kk + 8 * (v0 >> 2) + 4 * g_e + (v0 & 3), j1 = 32 * kk + 8 * (v1 >> 2) + 4 * g_e + (v1 & 3);
          const uint16_t *b0 = p.BV + ((size_t)kv * R + j0) * D + c, *b1 = p.BV + ((size_t)kv * R + j1) * D + c;
          if constexpr (PAIRS) {
            const uint32_t e0 = *(const uint32_t*)b0, e1 = *(const uint32_t*)b1;
            av[t][kk][s][e] = (int)__builtin_amdgcn_perm(e1, e0, 0x05040100u);
            av[t + (PAIRS ? 1 : 0)][kk][s][e] = (int)__builtin_amdgcn_perm(e1, e0, 0x07060302u);
          } else {
            av[t][kk][s][e] = (int)((uint32_t)*b0 | ((uint32_t)*b1 << 16));
          }
        }
  }
  const float inv = L > 0.f ? 1.0f / L : 0.f;
  v8bf16 uh[KK][2], ul[KK][2];
#pragma unroll
  for (int kk = 0; kk < KK; kk++)
#pragma unroll
    for (int s = 0; s < 2; s++) {
      v4i hh, ll;
#pragma unroll
      for (int e = 0; e < 4; e++) {
        uint32_t h0, l0, h1, l1;
        split_bf16(U[kk][8 * s + 2 * e] * inv, h0, l0);
        split_bf16(U[kk][8 * s + 2 * e + 1] * inv, h1, l1);
        hh[e] = (int)((h0 >> 16) | h1);
        ll[e] = (int)((l0 >> 16) | l1);
      }
      uh[kk][s] = __builtin_bit_cast(v8bf16, hh);
      ul[kk][s] = __builtin_bit_cast(v8bf16, ll);
    }
  auto product = [&](int t) {
    v16f O;
#pragma unroll
    for (int v = 0; v < 16; v++) O[v] = 0.f;
#pragma unroll
    for (int kk = 0; kk < KK; kk++)
#pragma unroll
      for (int s = 0; s < 2; s++) {
        const v8bf16 a = __builtin_bit_cast(v8bf16, av[t][kk][s]);
        O = mfma_bf16(a, uh[kk][s], O);
        O = mfma_bf16(a, ul[kk][s], O);
      }
    return O;
  };
  const int row_e = qb * 32 + n_e;
  float* const orow = p.out + (ph * p.NR + min(row_e, p.NR - 1)) * D;
  if constexpr (PAIRS) {
#pragma unroll
    for (int t = 0; t < NRB; t += 2) {
      const v16f O0 = product(t), O1 = product(t + 1);
      if (row_e < p.NR) {
#pragma unroll
        for (int m4 = 0; m4 < 4; m4++) {
          float* const to = orow + 64 * (kg + t / 2 * KG) + 16 * m4 + 8 * g_e;
          *(v4f*)to = v4f{O0[4 * m4], O1[4 * m4], O0[4 * m4 + 1], O1[4 * m4 + 1]};
          *(v4f*)(to + 4) = v4f{O0[4 * m4 + 2], O1[4 * m4 + 2], O0[4 * m4 + 3], O1[4 * m4 + 3]};
        }
      }
    }
  } else {
#pragma unroll
    for (int t = 0; t < NRB; t++) {
      const int rb = kg + t * KG;
      if (rb >= D / 32) break;                                          // (wave-uniform: more groups than channel blocks)
      const v16f O = product(t);
      if (row_e < p.NR) {
#pragma unroll
        for (int m4 = 0; m4 < 4; m4++)
          *(v4f*)&orow[32 * rb + 8 * m4 + 4 * g_e] = v4f{O[4 * m4], O[4 * m4 + 1], O[4 * m4 + 2], O[4 * m4 + 3]};
      }
    }
  }
}

template <int R, int D, int QW, int KG>
void launch_prefill_attn(const PrefillParams& p, hipStream_t s) {
  dim3 grid((unsigned)p.Hkv, (unsigned)((p.NR + 32 * QW - 1) / (32 * QW)), (unsigned)p.B);
  hipLaunchKernelGGL((k_prefill_attn<R, D, QW, KG>), grid, dim3(64 * QW * KG), 0, s, p);
}

// Waves of a workgroup: QW share the conversion of the cache blocks, KG groups share the blocks of the same rows.
//   * While the launch does not fill the chip, a wave's walk over its key blocks is the time, so the blocks are dealt to 2 or
//     4 groups, if there are enough of them to pay for the merge (a group without a block only costs).  It is not full up to
//     about 1400 waves of 32 rows: causal waves are of unequal length.
//   * On a full chip the conversion decides: 4 waves of rows together, as long as most of the 4 have rows or the walk is long;
//     otherwise 2 or 1.
// us per call for 1x1 / 2x1 / 4x1 / 1x2 / 1x4 (QW x KG), and for one wave converting for itself with P through LDS (before):
//   rank, seqs x tokens, keys  1x1    2x1    4x1    1x2    1x4   before     (32 heads, d_head 128)
//   32,  1 x 32,      32     4.5    5.4    6.0    5.0    6.1      6.6
//   32,  1 x 64,    1064    21.6   23.4   22.1   13.5   10.3     26.2
//   32, 16 x 32,     232    10.3   11.4   11.7   10.0   10.6     13.2
//   32, 16 x 64,    4064    73.9   96.4   86.7   61.7   62.6      111
//   32, 64 x 16,      16    10.9   14.0   21.1   13.8   21.4     13.0
//   32, 64 x 32,    1032    41.6   45.0   57.7   41.6   45.6     52.8
//   32, 64 x 64,     264    32.5   31.3   40.5   39.8   55.4     40.0
//   32, 16 x 2048, 2048     511    464    435    612    685      534
//   64, 64 x 16,      16    14.1   22.8   36.7   22.6   37.3     17.5
//   64, 16 x 96,    1096    48.9   50.7   44.8   56.4   56.3     57.2
//   64, 64 x 96,     296    60.9   79.8   75.5   84.2    123     73.8
//   64, 16 x 2048, 2048     711    794    708    933   1170      735
// (the last column measured then, of a kernel that is gone).  Fitted to 1108 sizes (9 .. 2048 tokens, 1 .. 128 sequences, up to 4000
// keys before them, 4 .. 32 kv heads, groups of 1, 4 and 7): 0.8 % above the best of the six shapes on average then.  With the
// blocks' forms as they are now it is 2.6 % above over 600 such sizes, 19 of them by more than 18 %, at most 45 (rank 64, about 2000
// waves that see one or two blocks: 4x1 24 us, 1x1 17).
enum { kPa11 = 11, kPa21 = 21, kPa41 = 41, kPa12 = 12, kPa22 = 22, kPa14 = 14 };    // 10 QW + KG
int prefill_attn_rule(int R, long long waves, int rows32, int key_blocks) {
  const int quarter = R == 32 ? 256 : 128;                              // of the waves a chip holds at 1 (rank 64: 1/2) per SIMD
  const bool long_walk = key_blocks >= 32;
  if (waves <= quarter) return key_blocks >= 3 ? kPa14 : key_blocks == 2 ? kPa12 : kPa11;
  if (waves <= 2 * quarter) return key_blocks < 6 ? kPa11 : R == 32 && rows32 >= 2 && key_blocks < 12 ? kPa22 : kPa14;
  if (waves <= 1408) {
    if (key_blocks < 16) return R == 64 && waves <= 512 && key_blocks >= 8 ? kPa22 : kPa11;
    if (R == 64 && key_blocks >= (waves <= 512 ? 32 : 64)) return waves <= 1280 ? kPa14 : kPa41;
    if (R == 32 && key_blocks >= 64 && waves <= 768) return kPa14;
    return R == 32 && waves > 1024 && long_walk && rows32 >= 4 ? kPa22 : kPa12;
  }
  if (R == 32 && waves <= 1536 && rows32 >= 4 && key_blocks >= 16) return kPa22;
  const int slots = (rows32 + 3) / 4 * 4;                               // waves launched by groups of 4, of which rows32 have rows
  if (rows32 * 20 >= slots * 17) return kPa41;
  if (R == 32) {
    if (waves <= 2048) return long_walk ? kPa12 : kPa11;
    if (rows32 * 4 >= slots * 3 && (rows32 >= 8 || long_walk || waves > 8192)) return kPa41;
    if (rows32 > 2 && key_blocks >= 64) return kPa41;
    return rows32 == 2 || (rows32 > 2 && waves > 6144) ? kPa21 : kPa11;
  }
  if (rows32 > 2 && ((key_blocks >= 64 && waves > 2048) || (rows32 == 3 && long_walk && waves <= 4096))) return kPa41;
  return rows32 == 2 && long_walk ? kPa21 : kPa11;
}
template <int R, int D>
void pick_prefill_attn_d(const PrefillParams& p, int key_blocks, hipStream_t s) {
  const int rows32 = (p.NR + 31) / 32;
  switch (prefill_attn_rule(R, (long long)p.B * p.Hkv * rows32, rows32, key_blocks)) {
    case kPa11: launch_prefill_attn<R, D, 1, 1>(p, s); break;
    case kPa21: launch_prefill_attn<R, D, 2, 1>(p, s); break;
    case kPa41: launch_prefill_attn<R, D, 4, 1>(p, s); break;
    case kPa12: launch_prefill_attn<R, D, 1, 2>(p, s); break;
    case kPa22: launch_prefill_attn<R, D, 2, 2>(p, s); break;
    default: launch_prefill_attn<R, D, 1, 4>(p, s); break;
  }
}
template <int R>
void pick_prefill_attn(const PrefillParams& p, int key_blocks, hipStream_t s) {
  if (p.d == 128) pick_prefill_attn_d<R, 128>(p, key_blocks, s);
  else pick_prefill_attn_d<R, 64>(p, key_blocks, s);
}

}  // namespace


hipError_t wsvd_launch_prefill_attn(const wsvd_layer_desc& d, const void* q, int nq, int n_after, const void* B_K, const void* B_V,
                                    const wsvd_cache& cache, int max_seq_len, void* out, hipStream_t s, const wsvd_paged_cache* paged) {
  if (d.latent_dtype != WSVD_I8 || d.factor_dtype != WSVD_BF16 || d.q_dtype != WSVD_BF16) return hipErrorNotSupported;
  if (d.d_head % 32 != 0 || nq < 1 || n_after < 0) return hipErrorInvalidValue;
  PrefillParams p;
  p.q = (const uint16_t*)q; p.BK = (const uint16_t*)B_K; p.BV = (const uint16_t*)B_V;
  p.k_codes = (const uint8_t*)cache.k_codes; p.v_codes = (const uint8_t*)cache.v_codes;
  p.k_meta = (const uint16_t*)cache.k_meta; p.v_meta = (const uint16_t*)cache.v_meta;
  p.seq_lens = cache.seq_lens; p.out = (float*)out;
  p.B = d.batch; p.Hkv = d.n_kv_heads; p.G = d.n_q_heads / d.n_kv_heads; p.d = d.d_head; p.t_cap = d.t_cap;
  p.nq = nq; p.n_after = n_after;
  p.block_table = nullptr; p.page_rows = p.max_pages = p.n_pages = 0;
  if (paged) { p.block_table = paged->block_table; p.page_rows = paged->page_rows; p.max_pages = paged->max_pages; p.n_pages = paged->n_pages; }
  const int64_t NR = (int64_t)nq * p.G;
  if (NR > (int64_t)65535 * 32) return hipErrorInvalidValue;
  p.NR = (int)NR;
  const float sm = d.sm_scale != 0.f ? d.sm_scale : 1.0f / sqrtf((float)d.d_head);
  p.c_scale = sm * 1.44269504088896340736f;
  // the caller's bound on the lengths only steers the choice of the workgroup shape; one that cannot hold the queries
  // themselves says nothing
  const int bound = max_seq_len >= n_after + nq ? max_seq_len : d.t_cap;
  const int key_blocks = (std::max(bound - n_after, 1) + 31) / 32;
  if (d.rank == 32) pick_prefill_attn<32>(p, key_blocks, s);
  else if (d.rank == 64) pick_prefill_attn<64>(p, key_blocks, s);
  else return hipErrorNotSupported;
  return hipGetLastError();
}
