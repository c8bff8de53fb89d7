// Decode attention over ONE shared rank-R latent per token with per-head up-projections: the conventional whole-matrix
// scheme the per-head method is contrasted with (Section 3.1, panel (b) of its figure; the "W/o per-head" variant of the
// latency appendix).  Built here in the form that suits the matrix cores: with the up-projection absorbed into the query,
// the 32 heads are the columns of a GEMM over the shared latent,
//     S [tokens x heads] = C_K [tokens x R] Q~^T [R x heads],     U^T [R x heads] += (diag(s_V) C_V)^T P [tokens x heads],
// so the latent stream is read ONCE for all heads (not once per head, as a per-head kernel run on the shared latent
// would), at the price of R-dimensional per-head queries and outputs: Q~_h = B_Kh q_h and o_h = B_Vh^T u_h move
// 2 * H * R * d factor elements per step where the per-head scheme moves 2 * H * r * d.
//   k_shared_absorb_limbs  Q~ [B, H, R] = (sm_scale log2 e) B_Kh q_h         bf16 MFMA, one wave per (head, 32 latent dims),
//                     as three 7-bit limbs of a unit per piece of the rank
//   k_shared_attn     per (sequence, split of its 128-token chunks, part of the value dims): scores on int8 MFMA (the cache
//                     codes are the A operand as stored; Q~ as three 7-bit limbs in LDS is the B operand), softmax down
//                     the head columns, value product on fp16 MFMA with each wave owning a quarter of the part's output
//                     dims; partial (m, l, U) per split
//   k_shared_out      merge of the splits, u = U / l, o_h = B_Vh^T u_h         vector ALU, one workgroup per (head, sequence)
// 32x32 accumulator layout throughout: lane L holds column L % 32, rows 8 (v / 4) + 4 (L / 32) + v % 4, v = 0..15.
#include <type_traits>

#include "wsvd_dev.h"
#include "wsvd_internal.h"

namespace {

constexpr int kSharedHeads = 32;          // the heads are the 32 columns of the products
constexpr int kSharedChunk = 128;         // tokens per workgroup pass: one 32-token block per wave
// A sequence's queries as limbs, [3][R / 32][64 lanes][16 B], and behind them the value of a unit, [piece][head] (at most
// 16 pieces).  The images lie an odd number of 256-byte pieces apart (the lanes of a store hold 32 sequences); the room for one is that of
// the same queries in fp32, 128 R bytes.
constexpr size_t shared_image_bytes(int R) { return (size_t)96 * R + 2304; }
static_assert(shared_image_bytes(256) <= 128 * 256, "the smallest rank's images fit");
constexpr float kLimbRange = 1040000.f;   // |Q~ / delta| stays below 2^20: three signed 7-bit limbs

typedef float v2f __attribute__((ext_vector_type(2)));
typedef int v2i_u __attribute__((ext_vector_type(2), aligned(2)));       // the K scales are aligned to their elements only

struct SharedParams {
  const uint16_t* q;          // bf16 [B, H, d]
  const uint16_t* BK;         // bf16 [H, R, d]
  const uint16_t* BV;
  const uint8_t* k_codes;     // [B][t_cap * R], 32-token blocks
  const uint8_t* v_codes;
  const uint16_t* k_scale;    // fp16 [B][t_cap]
  const uint16_t* v_scale;
  const int* seq_lens;
  uint8_t* qt;                // workspace: Q~ as limbs, [B] images
  float* pm;                  // workspace: partial running maxima [B, S, H]
  float* pl;                  //            partial sums           [B, S, H]
  float* pu;                  //            partial U              [B, S, H, R]
  float* out;                 // fp32 [B, H, d]
  int B, d, R, t_cap, S;
  int parts;                  // workgroups the value dims of the same tokens are divided over
  int per;                    // ranks above 1024: chunks of 128 tokens per split (at most 4)
  float c_scale;              // sm_scale * log2(e)
};

// ---------------------------------------------------------------- Q~ = c B_Kh q_h, as the score product reads it
// One workgroup per (head, piece of the rank, 32 sequences) holds that piece of Q~ in registers, so its maximum is known on
// the spot and the three signed 7-bit limbs of round(Q~ / delta) leave in the order of the int8 product's B operand:
// lane (head, g2) of step ks holds dims 32 ks + 16 g2 .. + 15.  A piece is a quarter of the rank up to 1024 and 256 dims
// above (the last one may be 128).  Every piece has its own delta: with one per head (32
// workgroups of 256 KB of factors each) the launch took 13.5 us at rank 1024.  Converted by every split's workgroup instead,
// the limbs cost 2800 vector instructions, 20 KB of code run once, before the first score.
template <int D, int NW>                                                // NW waves: a block of 32 dims each
__global__ __launch_bounds__(NW * 64) __attribute__((amdgpu_waves_per_eu(2, 4))) void k_shared_absorb_limbs(SharedParams p) {
  __shared__ float wmax[NW][32];
  const int lane = threadIdx.x & 63, wave = __builtin_amdgcn_readfirstlane(threadIdx.x >> 6), n = lane & 31, g2 = lane >> 5;
  const int h = blockIdx.x, piece = blockIdx.y, b = 32 * blockIdx.z + n, jb = piece * NW + wave, R = p.R;
  const bool past = 32 * jb >= R;                                       // a wave behind the last piece's end
  const uint16_t* qrow = p.q + ((size_t)min(b, p.B - 1) * kSharedHeads + h) * D + 8 * g2;
  const uint16_t* arow = p.BK + ((size_t)h * R + (past ? 0 : 32 * jb) + n) * D + 8 * g2;
  v8bf16 a[D / 16], x[D / 16];
#pragma unroll
  for (int ks = 0; ks < D / 16; ks++) { x[ks] = *(const v8bf16*)(qrow + 16 * ks); a[ks] = *(const v8bf16*)(arow + 16 * ks); }
  __builtin_amdgcn_sched_barrier(0);
  v16f acc;
#pragma unroll
  for (int v = 0; v < 16; v++) acc[v] = 0.f;
#pragma unroll
  for (int ks = 0; ks < D / 16; ks++) acc = mfma_bf16(a[ks], x[ks], acc);
  float amax = 0.f;
#pragma unroll
  for (int v = 0; v < 16; v++) {
    acc[v] *= p.c_scale;
    amax = fmaxf(amax, fabsf(acc[v]));
  }
  amax = fmaxf(amax, __shfl_xor(amax, 32));
  if (g2 == 0) wmax[wave][n] = past ? 0.f : amax;
  __syncthreads();
  float hm = 0.f;
#pragma unroll
  for (int w = 0; w < NW; w++) hm = fmaxf(hm, wmax[w][n]);
  const float delta = hm > 0.f ? hm / kLimbRange : 1.0f;                // value of one unit of the integer query
  const float inv_delta = 1.0f / delta;
  if (b >= p.B || past) return;
  uint8_t* image = p.qt + (size_t)b * shared_image_bytes(R);
  if (wave == 0 && g2 == 0) ((float*)(image + (size_t)96 * R))[piece * kSharedHeads + h] = delta;
  uint32_t w[3][4];                                                     // [limb][m4]: dims 8 m4 + 4 g2 .. + 3
#pragma unroll
  for (int m4 = 0; m4 < 4; m4++) {
    w[0][m4] = w[1][m4] = w[2][m4] = 0;
#pragma unroll
    for (int e = 0; e < 4; e++) {
      const int Q = (int)__builtin_rintf(acc[4 * m4 + e] * inv_delta);
      const int a0 = ((Q + 64) & 127) - 64, Q1 = (Q - a0) >> 7;         // Q = a0 + 128 Q1 exactly
      const int a1 = ((Q1 + 64) & 127) - 64, a2 = (Q1 - a1) >> 7;
      w[0][m4] |= ((uint32_t)a0 & 0xFFu) << (8 * e);
      w[1][m4] |= ((uint32_t)a1 & 0xFFu) << (8 * e);
      w[2][m4] |= ((uint32_t)a2 & 0xFFu) << (8 * e);
    }
  }
#pragma unroll
  for (int t = 0; t < 3; t++) {         // the two halves of the wave swap pieces: each keeps the 16 dims of its own half
    const uint32_t o0 = (uint32_t)__shfl_xor((int)(g2 ? w[t][0] : w[t][2]), 32);
    const uint32_t o1 = (uint32_t)__shfl_xor((int)(g2 ? w[t][1] : w[t][3]), 32);
    const v4i o = g2 ? v4i{(int)o0, (int)w[t][2], (int)o1, (int)w[t][3]} : v4i{(int)w[t][0], (int)o0, (int)w[t][1], (int)o1};
    *(v4i*)(image + (size_t)t * (32 * R) + jb * 1024 + (h + 32 * g2) * 16) = o;
  }
}

// ---------------------------------------------------------------- attention over the shared latent, all heads at once
// One workgroup per CU with one or two chunks of 128 tokens each: what bounds it beside the stream is what runs once, so code
// is short (the limbs come ready made) and every request leaves as early as registers allow.  16 sequences of 2048 rows,
// rank 1024 (67 MB): 34.5 -> 22.2 us; 1 of 8191 rows 36.2 -> 15.6; 64 of 2047 rows, rank 256 27.6 -> 19.8.
// LDS: limbs [3][R / 32][64 lanes][16 B], then 3 float tables [4 waves][32], P tiles [4 waves][32 heads][40] fp16, value
// scales [4 waves][128 tokens] fp16 (each wave its own copy).
template <int R, int VH>
__global__ __launch_bounds__(256) void k_shared_attn(SharedParams p) {
  constexpr int NKS = R / 32;             // 32-dim steps of the score contraction
  constexpr int NKK = R / VH / 128;       // 32-dim sub-blocks of the value dims one wave owns
  extern __shared__ __align__(16) uint8_t sh_lds[];
  v4i* limbs = (v4i*)sh_lds;                                            // [3][NKS][64]
  float* resc = (float*)(sh_lds + 3 * NKS * 1024);                      // [4][32] each: a head's rescaling of U,
  float* cmax = resc + 128;                                             // its maximum
  float* csum = cmax + 128;                                             // and its sum over a wave's tokens
  _Float16* pt = (_Float16*)(csum + 128);                               // [4][32][40]
  uint32_t* vsl = (uint32_t*)(pt + 4 * 32 * 40);                        // [4][64] pairs of fp16

  // (the wave's number in a scalar register: the planes' addresses are a scalar base and one offset per lane)
  const int tid = threadIdx.x, lane = tid & 63, wave = __builtin_amdgcn_readfirstlane(tid >> 6), n = lane & 31, g2 = lane >> 5;
  // workgroups go to the 8 dies in turn: the VH workgroups of the same tokens follow each other on one die, and so do the
  // splits of a sequence, which read the same limbs, where the sequences come in whole groups of 8
  const int unit = (blockIdx.x & 7) + 8 * (blockIdx.x / (8 * VH)), vh = (blockIdx.x >> 3) % VH;
  if (unit >= p.B * p.S) return;
  const int b = (p.B & 7) == 0 ? (unit & 7) + 8 * (unit / (8 * p.S)) : unit / p.S;
  const int split = (p.B & 7) == 0 ? (unit >> 3) % p.S : unit % p.S;
  const int n_b = min(max(p.seq_lens[b], 0), p.t_cap);
  const int n_chunks = (n_b + kSharedChunk - 1) / kSharedChunk;
  const int per = (n_chunks + p.S - 1) / p.S;
  const int c0 = split * per, c1 = min(c0 + per, n_chunks);
  const size_t part = (size_t)b * p.S + split;
  if (c0 >= c1) {                                                       // nothing for this split: the merge skips it
    if (tid < kSharedHeads) { p.pm[part * kSharedHeads + tid] = -INFINITY; p.pl[part * kSharedHeads + tid] = 0.f; }
    return;
  }

  const uint8_t* kplane = p.k_codes + (size_t)b * p.t_cap * R;
  const uint8_t* vplane = p.v_codes + (size_t)b * p.t_cap * R;
  const uint16_t* kmeta = p.k_scale + (size_t)b * p.t_cap;
  const uint16_t* vmeta = p.v_scale + (size_t)b * p.t_cap;

  // ---- the limbs of the sequence's queries, a quarter by each wave
  const uint8_t* qimage = p.qt + (size_t)b * shared_image_bytes(R);
  const v4i* image = (const v4i*)qimage + wave * (3 * NKS / 4) * 64 + lane;
  float delta[4];
#pragma unroll
  for (int i = 0; i < 4; i++) delta[i] = ((const float*)(qimage + 96 * R))[i * kSharedHeads + n];
  v4i lq[3 * NKS / 4];
#pragma unroll
  for (int i = 0; i < 3 * NKS / 4; i++) lq[i] = image[i * 64];
  // this wave's 32 tokens of a chunk: K scales of the accumulator's rows and all R / 32 operand blocks (and the V scales of
  // all 128 tokens).  The first chunk's
  // are requested here, behind the limbs
  v2i ksr[4];
  uint32_t vsr;
  const uint32_t lane16 = 16 * lane;
  v4i ka[NKS];
  const auto request_scales = [&](int c) {
#pragma unroll
    for (int m4 = 0; m4 < 4; m4++) ksr[m4] = *(const v2i_u*)(kmeta + c * kSharedChunk + 32 * wave + 8 * m4 + 4 * g2);
    vsr = *(const uint32_t*)(vmeta + c * kSharedChunk + 2 * lane);
  };
  const auto request_keys = [&](int c, int part4) {                     // a quarter of the chunk's blocks
    const uint8_t* kp = kplane + (size_t)(c * 4 + wave) * (32 * R);
#pragma unroll
    for (int ks = 0; ks < NKS / 4; ks++)
      {
      const v4i* src = (const v4i*)(kp + (part4 * (NKS / 4) + ks) * 1024 + lane16);
      ka[part4 * (NKS / 4) + ks] = VH > 1 ? *src : __builtin_nontemporal_load(src);
    }
  };
  request_scales(c0);
#pragma unroll
  for (int i = 0; i < 4; i++) request_keys(c0, i);
  __builtin_amdgcn_sched_barrier(0);
#pragma unroll
  for (int i = 0; i < 3 * NKS / 4; i++) limbs[(wave * (3 * NKS / 4) + i) * 64 + lane] = lq[i];
  __syncthreads();

  float m_run = -INFINITY, l_run = 0.f;                                 // of head n (every wave keeps its own copy)
  v16f U[NKK];                                                          // rows = heads, columns = this wave's dims
#pragma unroll
  for (int kk = 0; kk < NKK; kk++)
#pragma unroll
    for (int v = 0; v < 16; v++) U[kk][v] = 0.f;

  v4i vc[4][NKK];
  // One chunk: every quarter of the score product frees a quarter of the key registers and is followed by the requests of
  // one 32-token block of the values; every block of the value product is followed by the requests of a quarter of the
  // next chunk's keys.  So a whole plane's piece of the chunk (R x 128 bytes) is on its way at any time.
  const auto chunk = [&](int c, auto more) {
    const int cbase = c * kSharedChunk, t0 = cbase + 32 * wave;
    float sc[16];
#pragma unroll
    for (int tw = 0; tw < 4; tw++) {
      v16i a0, a1, a2;
#pragma unroll
      for (int v = 0; v < 16; v++) { a0[v] = 0; a1[v] = 0; a2[v] = 0; }
#pragma unroll
      for (int i = 0; i < NKS / 4; i++) {
        const int ks = tw * (NKS / 4) + i;
        a0 = mfma_i8(ka[ks], limbs[(0 * NKS + ks) * 64 + lane], a0);
        a1 = mfma_i8(ka[ks], limbs[(1 * NKS + ks) * 64 + lane], a1);
        a2 = mfma_i8(ka[ks], limbs[(2 * NKS + ks) * 64 + lane], a2);
        // keeps the limb reads from piling up in registers (rank 1024 in one part fills all 512: four steps' reads spill)
        if ((i & (NKK == 8 ? 1 : 3)) == (NKK == 8 ? 1 : 3)) __builtin_amdgcn_sched_barrier(0);
      }
      __builtin_amdgcn_sched_barrier(0);
      const int tv = min(cbase + 32 * tw, (n_b - 1) & ~31);             // (a block past the end: the last one again, unused)
      const uint8_t* vp = vplane + (size_t)(tv >> 5) * (32 * R) + (size_t)((4 * vh + wave) * NKK) * 1024;
#pragma unroll
      for (int kk = 0; kk < NKK; kk++) vc[tw][kk] = __builtin_nontemporal_load((const v4i*)(vp + kk * 1024 + lane16));
      __builtin_amdgcn_sched_barrier(0);
#pragma unroll
      for (int v = 0; v < 16; v++) {
        const float s = fmaf(16384.f, (float)a2[v], fmaf(128.f, (float)a1[v], (float)a0[v]));
        sc[v] = tw == 0 ? s * delta[0] : fmaf(s, delta[tw], sc[v]);
      }
    }
    float bmax = -INFINITY;
#pragma unroll
    for (int m4 = 0; m4 < 4; m4++) {
      const v4f k4 = __builtin_convertvector(__builtin_bit_cast(v4f16, ksr[m4]), v4f);
#pragma unroll
      for (int jj = 0; jj < 4; jj++) {
        const int v = 4 * m4 + jj;
        sc[v] = t0 + 8 * m4 + 4 * g2 + jj < n_b ? sc[v] * k4[jj] : -INFINITY;   // rows past the sequence's end
        bmax = fmaxf(bmax, sc[v]);
      }
    }
    bmax = fmaxf(bmax, __shfl_xor(bmax, 32));
    if (g2 == 0) cmax[wave * 32 + n] = bmax;
    __syncthreads();
    const float m_new = fmaxf(m_run, fmaxf(fmaxf(cmax[n], cmax[32 + n]), fmaxf(cmax[64 + n], cmax[96 + n])));
    const float alpha = m_run == -INFINITY ? 0.f : __builtin_amdgcn_exp2f(m_run - m_new);   // m_new is finite: the chunk has a row
    const bool rescale = c != c0 && __builtin_amdgcn_ballot_w64(alpha != 1.0f) != 0;        // (U is 0 at the first chunk)
    float pw[16], psum = 0.f;
#pragma unroll
    for (int v = 0; v < 16; v++) {
      pw[v] = sc[v] == -INFINITY ? 0.f : __builtin_amdgcn_exp2f(sc[v] - m_new);
      psum += pw[v];
    }
    psum += __shfl_xor(psum, 32);
    if (g2 == 0) { csum[wave * 32 + n] = psum; resc[wave * 32 + n] = alpha; }
    {                                     // rows never written may hold any scale: they contribute 0
      const int tl = cbase + 2 * lane;
      vsl[wave * 64 + lane] = tl + 1 < n_b ? vsr : tl < n_b ? vsr & 0xFFFFu : 0u;
    }
    _Float16* ptw = pt + (wave * 32 + n) * 40;
#pragma unroll
    for (int m4 = 0; m4 < 4; m4++) {
      v4f p4;
#pragma unroll
      for (int jj = 0; jj < 4; jj++) p4[jj] = pw[4 * m4 + jj];
      *(v2i*)&ptw[8 * m4 + 4 * g2] = __builtin_bit_cast(v2i, __builtin_convertvector(p4, v4f16));
    }
    __syncthreads();
    l_run = fmaf(l_run, alpha, (csum[n] + csum[32 + n]) + (csum[64 + n] + csum[96 + n]));
    m_run = m_new;
    if constexpr (decltype(more)::value) request_scales(c + 1);

    // ---- value product: this wave's quarter of the R dims, all four token blocks of the chunk
    if (rescale) {
#pragma unroll
      for (int m4 = 0; m4 < 4; m4++) {
        const v4f al = *(const v4f*)&resc[wave * 32 + 8 * m4 + 4 * g2];
#pragma unroll
        for (int kk = 0; kk < NKK; kk++)
#pragma unroll
          for (int jj = 0; jj < 4; jj++) U[kk][4 * m4 + jj] *= al[jj];
      }
    }
#pragma unroll
    for (int tw = 0; tw < 4; tw++) {
      const int tv = cbase + 32 * tw;
      if (tv < n_b) {
        const v8f16 sv0 = *(const v8f16*)&vsl[wave * 64 + 16 * tw + 8 * g2];
        const v8f16 sv1 = *(const v8f16*)&vsl[wave * 64 + 16 * tw + 8 * g2 + 4];
        const v8f16 bp0 = *(const v8f16*)&pt[(tw * 32 + n) * 40 + 16 * g2];
        const v8f16 bp1 = *(const v8f16*)&pt[(tw * 32 + n) * 40 + 16 * g2 + 8];
#pragma unroll
        for (int kk = 0; kk < NKK; kk++) {
          U[kk] = mfma_f16(bp0, codes_f16(vc[tw][kk][0], vc[tw][kk][1]) * sv0, U[kk]);
          U[kk] = mfma_f16(bp1, codes_f16(vc[tw][kk][2], vc[tw][kk][3]) * sv1, U[kk]);
        }
      }
      if constexpr (decltype(more)::value) {
        __builtin_amdgcn_sched_barrier(0);
        request_keys(c + 1, tw);
        __builtin_amdgcn_sched_barrier(0);
      }
    }
    if constexpr (decltype(more)::value) __syncthreads();               // the tables and P tiles are reused by the next chunk
  };
  for (int c = c0; c + 1 < c1; c++) chunk(c, std::true_type{});
  chunk(c1 - 1, std::false_type{});

  // ---- partial result of this split: a store instruction writes two heads' whole 128-byte lines (the heads as columns
  // made it 64 pieces of 16 bytes, 4 KB apart)
  if (vh == 0 && wave == 0 && g2 == 0) { p.pm[part * kSharedHeads + n] = m_run; p.pl[part * kSharedHeads + n] = l_run; }
  float* pu = p.pu + (part * kSharedHeads + 4 * g2) * R + (size_t)((4 * vh + wave) * NKK) * 32 + n;
#pragma unroll
  for (int v = 0; v < 16; v++)
#pragma unroll
    for (int kk = 0; kk < NKK; kk++) pu[(size_t)(8 * (v >> 2) + (v & 3)) * R + 32 * kk] = U[kk][v];
}

// ---------------------------------------------------------------- the same for ranks above 1024 (up to 4096)
// The query side of a rank this wide does not fit in LDS (3 limbs x R x 32 heads), and a wave's quarter of the value
// dims does not fit in registers, so both passes walk the latent in slabs of 1024 dims.  A workgroup owns up to NC
// chunks of 128 tokens.  Scores: for every slab the limbs of that slab are staged once and all the workgroup's chunks
// run against them, the integer dot products of a slab being added to a float score per (token, head).  Softmax: one
// maximum per head over all the workgroup's tokens (no running rescale), P kept in LDS as fp16.  Values: for every slab
// a wave accumulates its quarter of the slab's dims over all chunks and writes that piece of the partial result.
// The slabs of the value dims are divided over p.parts workgroups where that fills the chip; each computes the scores of all
// its tokens.  As above, what runs once is expensive, so the limbs come ready made, the value code is one chunk's
// (102 -> 50 KB of code) and a slab's keys are requested together, the first chunk's behind the limbs.  16 sequences of 600
// rows, rank 1920: 44.5 -> 28.1 us; 40 of 300 rows, rank 1280 38.2 -> 24.4; the launch for the heads' maxima is gone.
constexpr int kBigSlab = 1024;            // latent dims per slab
constexpr int kBigChunks = 4;             // chunks of 128 tokens per workgroup, at most

__global__ __launch_bounds__(256) void k_shared_attn_big(SharedParams p) {
  constexpr int NC = kBigChunks;
  constexpr int NKS = kBigSlab / 32;      // 32-dim steps of a full slab
  constexpr int NKK = kBigSlab / 128;     // 32-dim value blocks one wave owns in a full slab
  extern __shared__ __align__(16) uint8_t sh_lds[];
  v4i* limbs = (v4i*)sh_lds;                                            // [3][NKS][64]
  float* cmax = (float*)(sh_lds + 3 * NKS * 1024);                      // [4][32]
  float* csum = cmax + 128;                                             // [4][32]
  float* ksc = csum + 128;                                              // [NC][4][32]
  _Float16* pt = (_Float16*)(ksc + NC * 128);                           // [NC][4 token blocks][32 heads][40]

  const int tid = threadIdx.x, lane = tid & 63, wave = __builtin_amdgcn_readfirstlane(tid >> 6), n = lane & 31, g2 = lane >> 5;
  const int unit = (blockIdx.x & 7) + 8 * (blockIdx.x / (8 * p.parts)), part_v = (blockIdx.x >> 3) % p.parts;   // as above
  if (unit >= p.B * p.S) return;
  const int b = (p.B & 7) == 0 ? (unit & 7) + 8 * (unit / (8 * p.S)) : unit / p.S;
  const int split = (p.B & 7) == 0 ? (unit >> 3) % p.S : unit % p.S;
  const int R = p.R;
  const int n_b = min(max(p.seq_lens[b], 0), p.t_cap);
  const int n_chunks = (n_b + kSharedChunk - 1) / kSharedChunk;
  const int c0 = split * p.per, c1 = min(c0 + p.per, n_chunks);        // per <= NC by the launch's choice of splits
  const size_t part = (size_t)b * p.S + split;
  if (c0 >= c1) {                                                       // nothing for this split: the merge skips it
    if (tid < kSharedHeads) { p.pm[part * kSharedHeads + tid] = -INFINITY; p.pl[part * kSharedHeads + tid] = 0.f; }
    return;
  }
  const uint8_t* kplane = p.k_codes + (size_t)b * p.t_cap * R;
  const uint8_t* vplane = p.v_codes + (size_t)b * p.t_cap * R;
  const uint16_t* kmeta = p.k_scale + (size_t)b * p.t_cap;
  const uint16_t* vmeta = p.v_scale + (size_t)b * p.t_cap;
  const int n_slabs = (R + kBigSlab - 1) / kBigSlab;

  // K scales of this wave's 32 tokens of every chunk
#pragma unroll
  for (int c = 0; c < NC; c++)
    if (g2 == 0) ksc[(c * 4 + wave) * 32 + n] = c0 + c < c1 ? f16_bits_to_f32(kmeta[(c0 + c) * kSharedChunk + 32 * wave + n]) : 0.f;

  // ---- scores: sacc[c][v] = sum over the rank of (integer query of head n) . (codes of token row(v) of chunk c)
  float sacc[NC][16];
#pragma unroll
  for (int c = 0; c < NC; c++)
#pragma unroll
    for (int v = 0; v < 16; v++) sacc[c][v] = 0.f;
  const uint8_t* qimage = p.qt + (size_t)b * shared_image_bytes(R);
  const uint32_t lane16 = 16 * lane;
  for (int sl = 0; sl < n_slabs; sl++) {
    const int d0 = sl * kBigSlab;
    const int nks = min(kBigSlab, R - d0) >> 5;                         // a multiple of 4
    // this wave moves steps wave, wave + 4, ... of the slab's limbs; the keys of the first chunk are requested behind them
    v4i lq[NKS / 4][3], ka[NKS];
#pragma unroll
    for (int i = 0; i < NKS / 4; i++)
      if (4 * i < nks) {
#pragma unroll
        for (int t = 0; t < 3; t++)
          lq[i][t] = *(const v4i*)(qimage + (size_t)t * (32 * R) + (size_t)((d0 >> 5) + 4 * i + wave) * 1024 + lane16);
      }
    float delta[4];                                                     // of 256 dims each
#pragma unroll
    for (int i = 0; i < 4; i++)
      delta[i] = ((const float*)(qimage + (size_t)96 * R))[min((d0 >> 8) + i, (R - 1) >> 8) * kSharedHeads + n];
    const auto request_keys = [&](int c) {
      const uint8_t* kp = kplane + (size_t)((c0 + c) * 4 + wave) * (32 * (size_t)R) + (size_t)(d0 >> 5) * 1024;
#pragma unroll
      for (int k = 0; k < NKS; k += 4)
        if (k < nks) {
#pragma unroll
          for (int k1 = k; k1 < k + 4; k1++) ka[k1] = *(const v4i*)(kp + k1 * 1024 + lane16);
        }
    };
    request_keys(0);
    __builtin_amdgcn_sched_barrier(0);
    __syncthreads();                                                    // the previous slab's limbs are no longer read
#pragma unroll
    for (int i = 0; i < NKS / 4; i++)
      if (4 * i < nks) {
#pragma unroll
        for (int t = 0; t < 3; t++) limbs[(t * NKS + 4 * i + wave) * 64 + lane] = lq[i][t];
      }
    __syncthreads();
#pragma unroll
    for (int c = 0; c < NC; c++) {
      if (c0 + c < c1) {                                                // workgroup-uniform
        if (c > 0) request_keys(c);
#pragma unroll
        for (int g = 0; g < 4; g++) {                                   // 256 dims with a unit of their own
          if (8 * g < nks) {
            v16i a0, a1, a2;
#pragma unroll
            for (int v = 0; v < 16; v++) { a0[v] = 0; a1[v] = 0; a2[v] = 0; }
#pragma unroll
            for (int k4 = 8 * g; k4 < 8 * g + 8; k4 += 4) {
              if (k4 < nks) {
#pragma unroll
                for (int k = k4; k < k4 + 4; k++) {
                  a0 = mfma_i8(ka[k], limbs[(0 * NKS + k) * 64 + lane], a0);
                  a1 = mfma_i8(ka[k], limbs[(1 * NKS + k) * 64 + lane], a1);
                  a2 = mfma_i8(ka[k], limbs[(2 * NKS + k) * 64 + lane], a2);
                }
                __builtin_amdgcn_sched_barrier(0);                      // keeps the limb reads from piling up in registers
              }
            }
#pragma unroll
            for (int v = 0; v < 16; v++)
              sacc[c][v] = fmaf(fmaf(16384.f, (float)a2[v], fmaf(128.f, (float)a1[v], (float)a0[v])), delta[g], sacc[c][v]);
          }
        }
      }
    }
  }

  // ---- softmax over the workgroup's tokens: one maximum per head
  float bmax = -INFINITY;
#pragma unroll
  for (int c = 0; c < NC; c++) {
    const int t0 = (c0 + c) * kSharedChunk + 32 * wave;
#pragma unroll
    for (int m4 = 0; m4 < 4; m4++) {
      const v4f k4 = *(const v4f*)&ksc[(c * 4 + wave) * 32 + 8 * m4 + 4 * g2];
#pragma unroll
      for (int jj = 0; jj < 4; jj++) {
        const int v = 4 * m4 + jj;
        const float sv = sacc[c][v] * k4[jj];
        sacc[c][v] = (c0 + c < c1 && t0 + 8 * m4 + 4 * g2 + jj < n_b) ? sv : -INFINITY;   // rows past the sequence's end
        bmax = fmaxf(bmax, sacc[c][v]);
      }
    }
  }
  bmax = fmaxf(bmax, __shfl_xor(bmax, 32));
  if (g2 == 0) cmax[wave * 32 + n] = bmax;
  __syncthreads();
  const float m_all = fmaxf(fmaxf(cmax[n], cmax[32 + n]), fmaxf(cmax[64 + n], cmax[96 + n]));   // finite: chunk c0 has a row
  float psum = 0.f;
#pragma unroll
  for (int c = 0; c < NC; c++) {
    _Float16* ptw = pt + ((c * 4 + wave) * 32 + n) * 40;
#pragma unroll
    for (int m4 = 0; m4 < 4; m4++) {
      v4f p4;
#pragma unroll
      for (int jj = 0; jj < 4; jj++) {
        const float sv = sacc[c][4 * m4 + jj];
        p4[jj] = sv == -INFINITY ? 0.f : __builtin_amdgcn_exp2f(sv - m_all);
        psum += p4[jj];
      }
      *(v2i*)&ptw[8 * m4 + 4 * g2] = __builtin_bit_cast(v2i, __builtin_convertvector(p4, v4f16));
    }
  }
  psum += __shfl_xor(psum, 32);
  if (g2 == 0) csum[wave * 32 + n] = psum;
  __syncthreads();
  if (part_v == 0 && wave == 0 && g2 == 0) {
    p.pm[part * kSharedHeads + n] = m_all;
    p.pl[part * kSharedHeads + n] = (csum[n] + csum[32 + n]) + (csum[64 + n] + csum[96 + n]);
  }

  // ---- values: slab by slab, this wave's quarter of the slab's dims over all chunks
  for (int sl = part_v; sl < n_slabs; sl += p.parts) {
    const int d0 = sl * kBigSlab;
    const int nkk = min(kBigSlab, R - d0) >> 7;                         // 32-dim blocks per wave in this slab (1..8)
    const int blk0 = (d0 >> 5) + wave * nkk;                            // first 32-dim block of this wave
    v16f U[NKK];
#pragma unroll
    for (int kk = 0; kk < NKK; kk++)
#pragma unroll
      for (int v = 0; v < 16; v++) U[kk][v] = 0.f;
#pragma unroll 1
    for (int c = 0; c < c1 - c0; c++) {
      const int cbase = (c0 + c) * kSharedChunk;
      // all of the chunk's blocks of this slab are requested at once
      v4i vc[4][NKK], vsr[4][2];
#pragma unroll
      for (int tw = 0; tw < 4; tw++) {
        const int tv = min(cbase + 32 * tw, (n_b - 1) & ~31);         // (a block past the end: the last one again, unused)
        const uint8_t* vp = vplane + (size_t)(tv >> 5) * (32 * (size_t)R) + (size_t)blk0 * 1024;
#pragma unroll
        for (int kk = 0; kk < NKK; kk++)
          if (kk < nkk) vc[tw][kk] = __builtin_nontemporal_load((const v4i*)(vp + kk * 1024 + lane16));
        vsr[tw][0] = *(const v4i*)(vmeta + tv + 16 * g2);
        vsr[tw][1] = *(const v4i*)(vmeta + tv + 16 * g2 + 8);
      }
      __builtin_amdgcn_sched_barrier(0);
#pragma unroll
      for (int tw = 0; tw < 4; tw++) {
        const int tv = cbase + 32 * tw;
        if (tv < n_b) {
          v8f16 sv8[2] = {__builtin_bit_cast(v8f16, vsr[tw][0]), __builtin_bit_cast(v8f16, vsr[tw][1])};
          if (tv + 32 > n_b) {      // rows never written may hold any scale: they contribute 0
#pragma unroll
            for (int s2 = 0; s2 < 2; s2++)
#pragma unroll
              for (int e = 0; e < 8; e++)
                if (tv + 16 * g2 + 8 * s2 + e >= n_b) sv8[s2][e] = (_Float16)0;
          }
          const v8f16 bp0 = *(const v8f16*)&pt[((c * 4 + tw) * 32 + n) * 40 + 16 * g2];
          const v8f16 bp1 = *(const v8f16*)&pt[((c * 4 + tw) * 32 + n) * 40 + 16 * g2 + 8];
#pragma unroll
          for (int kk = 0; kk < NKK; kk++) {
            if (kk < nkk) {                                           // workgroup-uniform
              U[kk] = mfma_f16(bp0, codes_f16(vc[tw][kk][0], vc[tw][kk][1]) * sv8[0], U[kk]);
              U[kk] = mfma_f16(bp1, codes_f16(vc[tw][kk][2], vc[tw][kk][3]) * sv8[1], U[kk]);
            }
          }
        }
      }
    }
    float* pu = p.pu + (part * kSharedHeads + 4 * g2) * R + (size_t)blk0 * 32 + n;
#pragma unroll
    for (int kk = 0; kk < NKK; kk++) {
      if (kk < nkk) {
#pragma unroll
        for (int v = 0; v < 16; v++) pu[(size_t)(8 * (v >> 2) + (v & 3)) * R + 32 * kk] = U[kk][v];
      }
    }
  }
}

// ---------------------------------------------------------------- merge of the splits and o_h = B_Vh^T u_h
// One workgroup per (head, sequence): a head's factors are read by all sequences, from the L2 of one die (32 heads in turn
// over 8 dies).  What bounds it is the chain of memory trips, so the first partial results are requested before the weights
// of the splits are known, and registers are kept to 64 so that a CU holds 32 waves: 16 sequences of rank 1024, 8 splits,
// 10.1 us (16 splits, 256 threads with 4 trips for the partial results: 13.2).  Two or four sequences per workgroup read
// B_Vh less often, but with 150 to 250 registers no more than 8 waves fit a CU (64 sequences of rank 256: 9.7 -> 18 us).
template <int T>
__global__ __launch_bounds__(T) __attribute__((amdgpu_waves_per_eu(8))) void k_shared_out(SharedParams p) {
  constexpr int NR = T / 16;                                            // rows of B_Vh per step: 16 lanes of 8 channels each
  extern __shared__ __align__(16) uint8_t so_lds[];
  float* wn = (float*)so_lds;                                           // [32 splits]: weight of a split / total sum
  float* red = wn + 32;                                                 // [waves][128 channels]
  float* uT = red + T / 64 * 128;                                       // [R]
  const int tid = threadIdx.x, lane = tid & 63, wave = tid >> 6, h = blockIdx.x, b = blockIdx.y;
  float m = -INFINITY, l = 0.f;
  if (wave == 0 && lane < p.S) {                                        // lane s holds split s (at most 32)
    m = p.pm[((size_t)b * p.S + lane) * kSharedHeads + h];
    l = p.pl[((size_t)b * p.S + lane) * kSharedHeads + h];
  }
  const size_t sstride = (size_t)kSharedHeads * p.R;
  const float* pu = p.pu + (((size_t)b * p.S) * kSharedHeads + h) * p.R;
  v2f x[8];
  const auto request_partials = [&](int j, int s0) {                    // 8 loads of 8 bytes in flight
#pragma unroll
    for (int i = 0; i < 8; i++) x[i] = *(const v2f*)(pu + min(s0 + i, p.S - 1) * sstride + j);
  };
  if (2 * tid < p.R) request_partials(2 * tid, 0);
  __builtin_amdgcn_sched_barrier(0);
  if (wave == 0) {
    const float M = wave_max(m);
    const float e = m == -INFINITY ? 0.f : __builtin_amdgcn_exp2f(m - M);
    const float L = wave_sum(e * l);
    if (lane < 32) wn[lane] = L > 0.f ? e / L : 0.f;                    // (past the last split: 0)
  }
  __syncthreads();
  for (int j = 2 * tid; j < p.R; j += 2 * T) {
    v2f u = {0.f, 0.f};
    for (int s0 = 0; s0 < p.S; s0 += 8) {
      if (j >= 2 * T || s0 > 0) request_partials(j, s0);
      const v4f wa = *(const v4f*)&wn[s0], wb = *(const v4f*)&wn[s0 + 4];
#pragma unroll
      for (int i = 0; i < 8; i++) {                                     // a split that wrote nothing has weight 0 and its
        const float ws = i < 4 ? wa[i & 3] : wb[i & 3];                 // (unwritten) values are dropped
        u[0] += ws != 0.f ? ws * x[i][0] : 0.f;
        u[1] += ws != 0.f ? ws * x[i][1] : 0.f;
      }
    }
    *(v2f*)&uT[j] = u;
  }
  __syncthreads();
  // thread (c8, js): output channels 8 c8 .. + 7 (one 16-byte load per row of B_Vh) of rows js, js + NR, ...
  const int c8 = tid & 15, js = tid >> 4;
  float acc[8];
#pragma unroll
  for (int e = 0; e < 8; e++) acc[e] = 0.f;
  if (8 * c8 < p.d) {
    const uint16_t* bv = p.BV + ((size_t)h * p.R + js) * p.d + 8 * c8;
    const auto rows = [&](int j, auto count) {                          // `count` loads in flight
      constexpr int N = decltype(count)::value;
      v4i w[N];
#pragma unroll
      for (int i = 0; i < N; i++) w[i] = *(const v4i*)(bv + (size_t)(j + i * NR) * p.d);
#pragma unroll
      for (int i = 0; i < N; i++) {
        const float u = uT[j + i * NR + js];
#pragma unroll
        for (int e2 = 0; e2 < 4; e2++) {
          acc[2 * e2] = fmaf(u, __uint_as_float((uint32_t)w[i][e2] << 16), acc[2 * e2]);
          acc[2 * e2 + 1] = fmaf(u, __uint_as_float((uint32_t)w[i][e2] & 0xFFFF0000u), acc[2 * e2 + 1]);
        }
      }
    };
    int j = 0;
    for (; j + 8 * NR <= p.R; j += 8 * NR) rows(j, std::integral_constant<int, 8>{});
    for (; j < p.R; j += NR) rows(j, std::integral_constant<int, 1>{});
  }
#pragma unroll
  for (int e = 0; e < 8; e++) {                                         // the wave's 4 rows of a step
    acc[e] += __shfl_xor(acc[e], 16);
    acc[e] += __shfl_xor(acc[e], 32);
  }
  if (lane < 16 && 8 * c8 < p.d) {
#pragma unroll
    for (int e = 0; e < 8; e++) red[wave * 128 + 8 * c8 + e] = acc[e];
  }
  __syncthreads();
  if (tid < p.d) {
    float o = 0.f;
#pragma unroll
    for (int q = 0; q < T / 64; q++) o += red[q * 128 + tid];
    p.out[((size_t)b * kSharedHeads + h) * p.d + tid] = o;
  }
}

// Workgroups over which the value dims of the same tokens are divided (each computes the scores of all its tokens), up to
// rank 1024.  Where (sequence, chunk) pairs are too few for the chip the parts fill it (1 sequence of 8191 rows, rank 1024:
// 1 / 2 / 4 parts 23.7 / 17.5 / 15.6 us; 5 of 3000 rows, rank 512: 10.8 / 8.8 us).  At rank 1024 two parts still pay with about one
// pair per workgroup: they halve the partial results, 33.6 MB at 16 sequences of 2048 rows, for a second reading of the keys
// from the die's cache.  With more pairs the second score pass costs more than that.  us per call, one part / two: rank 1024, 16 x
// 2048 rows 42 / 40, 20 x 2048 50 / 47, 33 x 2048 64 / 71, 65 x 2048 103 / 125, 64 x 8192 213 / 297; rank 512, 9 x 2048 rows 21.8 / 23.2,
// 5 x 4000 21.0 / 23.4; rank 256, 9 x 2048 17.3 / 18.1.  Not for 65 to 85 sequences, which have three splits in one part and one
// in two (65 of 300 rows, rank 1024, 62 / 65), nor beyond 128 (129 of 300 rows 103 / 120).
int shared_value_parts(int batch, int chunks, int rank) {
  const long pairs = (long)batch * chunks, splits = (long)batch * (chunks < 32 ? chunks : 32);    // (a sequence has at most 32)
  if (rank >= 512 && 4 * splits <= 256) return 4;
  return 2 * splits <= 256 || (rank == 1024 && pairs <= 320 && batch <= 128 && 256 / batch != 3) ? 2 : 1;
}

// Splits of a sequence then: as many as fit the CUs, one more would be a second round (65 x 2048 rows, rank 1024: three 103 us,
// four 130).  At rank 256 two workgroups fit a CU, so that from 129 sequences on two splits are still one round (129 x 2048
// rows: 80 -> 69 us).
int shared_splits_run(int batch, int parts, int rank, int most) {
  int s = 256 / (batch * parts);
  if (rank == 256 && parts == 1 && s == 1 && batch < 256) s = 2;
  return s < 1 ? 1 : s < most ? s : most;                               // never more than the workspace is sized for
}

int shared_splits(int batch, int t_cap, int rank) {
  int s = (256 + batch - 1) / batch;
  const int chunks = (t_cap + kSharedChunk - 1) / kSharedChunk;
  if (s > chunks) s = chunks;
  // ranks above 1024: a workgroup holds the scores of at most kBigChunks chunks
  if (rank > 1024 && s < (chunks + kBigChunks - 1) / kBigChunks) s = (chunks + kBigChunks - 1) / kBigChunks;
  if (s > 32) s = 32;
  return s < 1 ? 1 : s;
}

}  // namespace

// The launch's plan.  (The workspace is sized for shared_splits, which no plan exceeds.)  Above rank 1024 as many parts as fit the
// chip at once: 2 sequences of 1500 rows, rank 3712, 1 / 2 / 4 parts 56.6 / 45.3 / 39.2 us; 16 of 600 rows, rank 1920 (80
// workgroups), 33.5 / 28.1; with more than 256 workgroups there are two rounds (parts of nothing there: 49).
void wsvd_shared_plan(int batch, int rank, int t_cap, int* splits, int* parts) {
  const int most = shared_splits(batch, t_cap, rank), chunks = (t_cap + kSharedChunk - 1) / kSharedChunk;
  if (rank > 1024) {
    *splits = most;
    *parts = max(1, min(256 / (batch * most), (rank + kBigSlab - 1) / kBigSlab));
  } else {
    *parts = shared_value_parts(batch, chunks, rank);
    *splits = shared_splits_run(batch, *parts, rank, most);
  }
}

size_t wsvd_shared_ws_bytes(int batch, int rank, int t_cap) {
  const size_t S = (size_t)shared_splits(batch, t_cap, rank);
  const size_t floats = (size_t)batch * kSharedHeads * rank + 2 * (size_t)batch * S * kSharedHeads + (size_t)batch * S * kSharedHeads * rank;
  return floats * sizeof(float);
}

hipError_t wsvd_launch_attn_shared(int batch, int d_head, int rank, int t_cap, float sm_scale, const void* q, const void* B_K,
                                   const void* B_V, const void* k_codes, const void* v_codes, const void* k_scale,
                                   const void* v_scale, const int* seq_lens, void* workspace, void* out, hipStream_t s) {
  SharedParams p;
  p.q = (const uint16_t*)q; p.BK = (const uint16_t*)B_K; p.BV = (const uint16_t*)B_V;
  p.k_codes = (const uint8_t*)k_codes; p.v_codes = (const uint8_t*)v_codes;
  p.k_scale = (const uint16_t*)k_scale; p.v_scale = (const uint16_t*)v_scale;
  p.seq_lens = seq_lens;
  p.B = batch; p.d = d_head; p.R = rank; p.t_cap = t_cap;
  wsvd_shared_plan(batch, rank, t_cap, &p.S, &p.parts);
  const int chunks_cap = (t_cap + kSharedChunk - 1) / kSharedChunk;
  p.per = (chunks_cap + p.S - 1) / p.S;
  if (rank > 1024 && (p.per > kBigChunks || rank % 128 != 0 || rank > 4096)) return hipErrorNotSupported;
  p.c_scale = sm_scale * 1.4426950408889634f;
  p.qt = (uint8_t*)workspace;                                           // 128 R bytes for each of the images
  p.pm = (float*)workspace + (size_t)batch * kSharedHeads * rank;
  p.pl = p.pm + (size_t)batch * p.S * kSharedHeads;
  p.pu = p.pl + (size_t)batch * p.S * kSharedHeads;
  p.out = (float*)out;

  if (d_head != 64 && d_head != 128) return hipErrorNotSupported;
  const int waves_a = rank > 1024 ? 8 : rank / 128;
  const dim3 grid_a(kSharedHeads, (unsigned)((rank / 32 + waves_a - 1) / waves_a), (unsigned)((batch + 31) / 32));
  void (*fn_a)(SharedParams) = waves_a == 2   ? (d_head == 128 ? k_shared_absorb_limbs<128, 2> : k_shared_absorb_limbs<64, 2>)
                               : waves_a == 4 ? (d_head == 128 ? k_shared_absorb_limbs<128, 4> : k_shared_absorb_limbs<64, 4>)
                                              : (d_head == 128 ? k_shared_absorb_limbs<128, 8> : k_shared_absorb_limbs<64, 8>);
  hipLaunchKernelGGL(fn_a, grid_a, dim3((unsigned)waves_a * 64), 0, s, p);
  hipError_t e = hipGetLastError();
  if (e != hipSuccess) return e;

  // 512 threads shorten the chain of trips (1 sequence, rank 1024: 7.6 us, 256 threads 11.6; 2 of rank 3712: 17.5, 27.6);
  // at rank 256 half of them have no partial result to read (64 sequences: 10.7, 256 threads 8.4)
  const int t_out = rank == 256 ? 256 : 512;
  const size_t lds_out = (size_t)(32 + t_out / 64 * 128 + rank) * sizeof(float);       // at most 21 KB
  void (*fn_out)(SharedParams) = t_out == 512 ? k_shared_out<512> : k_shared_out<256>;
  const dim3 grid_out(kSharedHeads, (unsigned)batch);
  if (rank > 1024) {
    const size_t lds_big = (size_t)3 * (kBigSlab / 32) * 1024 + (size_t)(2 + kBigChunks) * 128 * sizeof(float) +
                           (size_t)kBigChunks * 4 * 32 * 40 * sizeof(_Float16);
    static LdsLimit limit_big;
    e = wsvd_raise_lds(limit_big, (const void*)k_shared_attn_big, (int)lds_big);
    if (e != hipSuccess) return e;
    hipLaunchKernelGGL(k_shared_attn_big, dim3((unsigned)((batch * p.S + 7) / 8 * 8 * p.parts)), dim3(256), lds_big, s, p);
    e = hipGetLastError();
    if (e != hipSuccess) return e;
    hipLaunchKernelGGL(fn_out, grid_out, dim3((unsigned)t_out), lds_out, s, p);
    return hipGetLastError();
  }
  const size_t lds_attn = (size_t)3 * (rank / 32) * 1024 + 3 * 128 * sizeof(float) +
                          4 * 32 * 40 * sizeof(_Float16) + 4 * 128 * sizeof(_Float16);
  const int vh = p.parts;
  void (*fn)(SharedParams) = rank == 256   ? (vh == 2 ? k_shared_attn<256, 2> : k_shared_attn<256, 1>)
                             : rank == 512 ? (vh == 4 ? k_shared_attn<512, 4> : vh == 2 ? k_shared_attn<512, 2> : k_shared_attn<512, 1>)
                                           : (vh == 4 ? k_shared_attn<1024, 4> : vh == 2 ? k_shared_attn<1024, 2> : k_shared_attn<1024, 1>);
  static LdsLimit limit[3];                                             // of the three kernels of rank 1024 (109 KB)
  if (rank == 1024) {
    e = wsvd_raise_lds(limit[vh >> 1], (const void*)fn, (int)lds_attn);
    if (e != hipSuccess) return e;
  }
  hipLaunchKernelGGL(fn, dim3((unsigned)((batch * p.S + 7) / 8 * 8 * vh)), dim3(256), lds_attn, s, p);
  e = hipGetLastError();
  if (e != hipSuccess) return e;

  hipLaunchKernelGGL(fn_out, grid_out, dim3((unsigned)t_out), lds_out, s, p);
  return hipGetLastError();
}
