// Cache build for a whole prompt (the projection of prefilling, Section 3.4): C = x A for all prompt tokens on the matrix
// cores, per-token int8 quantisation and stores in the decode layout.
#include "wsvd_dev.h"
#include "wsvd_internal.h"

namespace {

// ---------------------------------------------------------------- cache build for a whole prompt (int8 latents)
// C^T [channels x tokens] = A^T x^T on bf16 MFMA.  The channels of both planes form one axis of 2 * Hkv * r / 32 tiles
// of 32; a wavefront owns CT channel tiles x TT token tiles (CT * TT accumulators of 32 x 32), so each 1 KiB operand it
// fetches feeds CT or TT products.  The A operand is the packed factor image the append kernels use (1 KiB per
// 32 channels x 16 model dims, contiguous); the B operand is 16 bytes of a token's hidden state per lane.  The 4 waves
// of a workgroup take 4 neighbouring channel groups of the same tokens, so the hidden states come out of the CU's
// first-level cache after the first wave; operands are requested ST - 1 steps ahead of the products that use them.
// A lane ends up with 16 of every 32 channels of ITS tokens (the other half wave holds the rest): the per-token scale of
// a head is a maximum over registers plus one exchange, and the codes go out in the decode layout (4 consecutive
// channels of a K row are 4 adjacent bytes; a V row is written byte by byte, its neighbours in a 16-byte group being
// other tokens).
struct ProjectParams {
  const uint16_t* x;          // bf16 [n_seq, n_tok, E]
  const uint16_t* A[2];       // packed factors
  uint8_t* codes[2];
  uint16_t* meta[2];
  int* seq_lens;
  int* err_word;
  int Hkv, E, t_cap, n_tok, seq0;   // direct kernel: grid z = sequence - seq0
  int rows;                         // rows that tiles are cut from: n_tok, or n_seq * n_tok (tiles across sequences)
  int n_cg, tg_seq, n_tg;           // tile kernels: channel groups, token groups per set of rows and in all
  bool token_affine;                // tile kernels: see project_groups
  // paged cache only (else null): codes / meta are pools of n_pages pages, a page = page_rows rows of every kv head in the
  // layout of a contiguous plane; block_table [B][max_pages]
  const int* block_table;
  int page_rows, max_pages, n_pages;
  // tile kernels: workgroups of this launch that hold the lengths they need (the context's counter, zero between launches), and
  // what the last of them advances
  int* readers;
  int n_seq, even_only;
};

// The lengths move on by the rows that fitted (sequence i of the call).  int4: nothing was stored for a sequence that starts on
// an odd row.
WSVD_DEV void project_bump(int* seq_lens, int i, int n_tok, int t_cap, int* err_word, int even_only) {
  const int n0 = seq_lens[i];
  if (even_only && n0 >= 0 && (n0 & 1)) {
    atomicExch(err_word, (int)WSVD_E_SHAPE);
    return;
  }
  if (n0 >= 0) seq_lens[i] = min(n0 + n_tok, t_cap);
  if (n0 < 0 || n0 + n_tok > t_cap) atomicExch(err_word, (int)WSVD_E_CAPACITY);
}
// The tile kernels advance the lengths themselves: every workgroup counts itself once all its waves hold the lengths they store
// by (the barrier in front), asks for the count so far, and looks at the answer when its rows are stored; the last one to
// have counted advances them.  Eight counters a line apart, and one for whoever fills one of them: on a single word 512
// workgroups that end together waited for each other's additions, 0.7 us.  2 x 35 tokens 15.5 -> 14.5 us, 1 x 200 15.8 -> 15.1,
// 3 x 333 30.7 -> 29.4 (32 heads of rank 32, with the clearing of the lengths before it).
constexpr int kReaderGap = 32;                                           // ints between two counters
template <int N>
WSVD_DEV void project_hold(const int (&n0)[N]) {                         // the lengths are here (in front of a barrier)
#pragma unroll
  for (int i = 0; i < N; i++) asm volatile("" ::"v"(n0[i]) : "memory");
}
WSVD_DEV int project_count(const ProjectParams& p) {
  int seen = -1;
  if (threadIdx.x == 0) seen = __hip_atomic_fetch_add(p.readers + kReaderGap * (1 + (blockIdx.x & 7)), 1, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT);
  return seen;
}
WSVD_DEV void project_advance(const ProjectParams& p, int seen) {        // seen: of the workgroup's first lane; waves 1.. hold -1
  const int n = (int)gridDim.x, g = (int)(blockIdx.x & 7);
  if (__builtin_amdgcn_readfirstlane(seen) != (n + 7 - g) / 8 - 1) return;
  const int lane = lane_number();
  int last = 0;
  if (lane == 0) {
    __hip_atomic_store(p.readers + kReaderGap * (1 + g), 0, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT);
    last = __hip_atomic_fetch_add(p.readers, 1, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT) == min(n, 8) - 1;
    if (last) __hip_atomic_store(p.readers, 0, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT);
  }
  if (__builtin_amdgcn_readfirstlane(last) == 0) return;
  for (int i = lane; i < p.n_seq; i += 64) project_bump(p.seq_lens, p.seq0 + i, p.n_tok, p.t_cap, p.err_word, p.even_only);
}

// Where row t of (sequence, kv head) lives: its plane (row_bytes per row), its row inside that plane, the index of its
// metadata entry.  Paged: a table entry outside the pools is reported and the row is not stored (ok = false).
struct ProjRow { uint8_t* plane; size_t meta; int t; bool ok; };
WSVD_DEV ProjRow project_row(const ProjectParams& p, int pl, int seq, int kv, int t, int row_bytes) {
  ProjRow r;
  if (!p.block_table) {
    const size_t ph = (size_t)seq * p.Hkv + kv;
    r.plane = p.codes[pl] + ph * (size_t)p.t_cap * row_bytes; r.meta = ph * p.t_cap + t; r.t = t; r.ok = true;
    return r;
  }
  const int pg = min(max(t, 0) / p.page_rows, p.max_pages - 1);
  const int e = p.block_table[(size_t)seq * p.max_pages + pg];
  r.ok = e >= 0 && e < p.n_pages;
  if (!r.ok) atomicExch(p.err_word, (int)WSVD_E_SHAPE);
  const size_t slot = (size_t)(r.ok ? e : 0) * p.Hkv + kv;
  r.t = t - pg * p.page_rows;
  r.plane = p.codes[pl] + slot * (size_t)p.page_rows * row_bytes;
  r.meta = slot * p.page_rows + r.t;
  return r;
}

// One token's row of one head and plane: the 16 channels of every 32 that this lane holds in a[], the rest in its partner
// half.  Symmetric int8 (the latent quantiser's rule), then the stores.  The codes are made without a branch, so that those of
// several rows can overlap (4 waves of 16 such rows each: 17 us one after the other, 14 four at a time).
template <int RT>
struct RowI8 {
  uint32_t codes[RT][4];                                                // channels 32 rt + 8 m4 + 4 g2 .. + 3
  uint16_t scale;
};
template <int RT>
WSVD_DEV RowI8<RT> quantise_row_i8(const v16f (&a)[RT]) {
  RowI8<RT> r;
  float m = 0.f;
#pragma unroll
  for (int rt = 0; rt < RT; rt++)
#pragma unroll
    for (int v = 0; v < 16; v++) m = fmaxf(m, fabsf(a[rt][v]));
  m = halves_max(m);
  r.scale = m != 0.f ? guard_scale_f16(m / 127.0f) : (uint16_t)0x3C00u;
  const float sc = f16_bits_to_f32(r.scale), inv = 1.0f / sc;
#pragma unroll
  for (int rt = 0; rt < RT; rt++)
#pragma unroll
    for (int m4 = 0; m4 < 4; m4++) {
      uint32_t pk = 0;
#pragma unroll
      for (int jj = 0; jj < 4; jj++) {
        const int q = (int)__builtin_amdgcn_fmed3f(__builtin_rintf(div_by_scale(a[rt][4 * m4 + jj], sc, inv)), -127.f, 127.f);
        pk |= ((uint32_t)q & 0xFFu) << (8 * jj);
      }
      r.codes[rt][m4] = pk;
    }
  return r;
}
template <int RT>
WSVD_DEV void put_row_i8(const ProjectParams& p, const RowI8<RT>& r, int pl, int seq, int kv, int t, bool on) {
  constexpr int R = 32 * RT;
  const int g2 = lane_number() >> 5;
  if (!on) return;
  const ProjRow pr = project_row(p, pl, seq, kv, t, R);
  if (!pr.ok) return;
#pragma unroll
  for (int rt = 0; rt < RT; rt++)
#pragma unroll
    for (int m4 = 0; m4 < 4; m4++) {
      const int j0 = 32 * rt + 8 * m4 + 4 * g2;                         // channels j0 .. j0 + 3
      const uint32_t pk = r.codes[rt][m4];
      if (pl == 0) *(uint32_t*)(pr.plane + i8_k_offset(pr.t, j0, R)) = pk;
      else {
#pragma unroll
        for (int jj = 0; jj < 4; jj++) pr.plane[i8_v_offset(pr.t, j0 + jj, R)] = (uint8_t)(pk >> (8 * jj));
      }
    }
  if (g2 == 0) p.meta[pl][pr.meta] = r.scale;
}

// The same for int4 (rank 32: one channel tile per head): the rule of quantize_row_i4; K bytes pair dims (2 adjacent
// registers), V bytes pair rows t, t ^ 1 = this lane and its neighbour (the caller guarantees an even start row, so row
// parity = lane parity).  next_on: the neighbour's row is stored too.
WSVD_DEV void store_row_i4(const ProjectParams& p, const v16f& a, int pl, int seq, int kv, int t, bool on, bool next_on) {
  const int lane = lane_number(), g2 = lane >> 5;
  float lo = 0.f, hi = 0.f;
#pragma unroll
  for (int v = 0; v < 16; v++) { lo = fminf(lo, a[v]); hi = fmaxf(hi, a[v]); }
  lo = -halves_max(-lo); hi = halves_max(hi);
  uint16_t sh = 0x3C00u;
  float z = 0.f;
  const bool flat = (hi == lo);
  if (!flat) sh = guard_scale_f16((hi - lo) / 15.0f);
  const float sc = f16_bits_to_f32(sh), inv = 1.0f / sc;
  if (!flat) z = fminf(fmaxf(__builtin_rintf(-lo / sc), 0.f), 15.f);
  const int zi = (int)z;
  ProjRow pr = {nullptr, 0, t, false};
  if (on) { pr = project_row(p, pl, seq, kv, t, 16); on = pr.ok; }
#pragma unroll
  for (int m4 = 0; m4 < 4; m4++) {
    int q[4];
#pragma unroll
    for (int jj = 0; jj < 4; jj++) {
      const float v = fminf(fmaxf(__builtin_rintf(div_by_scale(a[4 * m4 + jj], sc, inv)), -64.f), 64.f);
      const int qq = (int)v + zi;
      q[jj] = qq < 0 ? 0 : (qq > 15 ? 15 : qq);
    }
    const int j0 = 8 * m4 + 4 * g2;                                     // channels j0 .. j0 + 3
    int nib;
    if (pl == 0) {
      if (on) *(uint16_t*)(pr.plane + i4_k_offset(pr.t, j0, &nib)) = (uint16_t)(q[0] | (q[1] << 4) | (q[2] << 8) | (q[3] << 12));
    } else {
#pragma unroll
      for (int jj = 0; jj < 4; jj++) {
        const int qn = __builtin_amdgcn_update_dpp(0, q[jj], kDppQuadSwap1, 0xF, 0xF, true);   // the neighbour row's code
        if (on && (lane & 1) == 0) pr.plane[i4_v_offset(pr.t, j0 + jj, &nib)] = (uint8_t)(q[jj] | ((next_on ? qn : 0) << 4));
      }
    }
  }
  if (on && g2 == 0) *(uint32_t*)&p.meta[pl][pr.meta * 2] = (uint32_t)sh | ((uint32_t)f32_to_f16_bits_rne((float)zi) << 16);
}

// acc[c][tt] = channel tile ct0 + c x token tile tb * TT + tt of this wave, in the 32 x 32 accumulator order.  The format
// is a template parameter and no loop leaves early: every index into acc has to be a constant after unrolling.  (With
// both formats in one body the loops stayed rolled, acc was indexed at run time and all 256 accumulators of a lane lived
// in scratch memory: 10.2 ms for 16 x 2048 tokens against 0.5 ms.)
// SPAN: a tile's rows run on into the next sequences (row % n_tok of sequence seq + row / n_tok); otherwise all are of
// sequence seq.  n0: the rows that a row's sequence holds, asked for ahead of the store.
template <bool SPAN>
WSVD_DEV int row_length(const ProjectParams& p, int seq, int row) {
  return p.seq_lens[SPAN ? seq + min(row, p.rows - 1) / p.n_tok : seq];
}
// Tiles [tt0, tt0 + N) of head h of the wave.
template <int R, int CT, int TT, bool I4, bool SPAN, int N>
WSVD_DEV void project_store_tiles(const ProjectParams& p, const v16f (&acc)[CT][TT], int h, int tt0, int ct0, int row0, int seq, const int (&n0)[TT]) {
  constexpr int RT = R / 32;
  static_assert(!I4 || R == 32, "int4 latents have rank 32");
  const int tiles_plane = p.Hkv * RT, tiles = 2 * tiles_plane;
  const int ct = ct0 + h * RT;
  const int pl = ct >= tiles_plane, kv = (ct - (pl ? tiles_plane : 0)) / RT;   // (wave-uniform; no division: its reciprocal was kept)
  RowI8<RT> rows[N];
  if constexpr (!I4) {
#pragma unroll
    for (int i = 0; i < N; i++) {
      v16f a[RT];
#pragma unroll
      for (int rt = 0; rt < RT; rt++) a[rt] = acc[h * RT + rt][tt0 + i];
      rows[i] = quantise_row_i8<RT>(a);
    }
  }
#pragma unroll
  for (int i = 0; i < N; i++) {
    const int tt = tt0 + i;
    const int row = row0 + 32 * tt + (lane_number() & 31), sq = SPAN ? min(row, p.rows - 1) / p.n_tok : 0;
    const int tok = row - sq * p.n_tok, t = n0[tt] + tok;               // this lane's token of the prompt, its cache row
    const bool on = ct < tiles && row < p.rows && n0[tt] >= 0 && t < p.t_cap;
    if constexpr (I4) store_row_i4(p, acc[h][tt], pl, seq + sq, kv, t, on && (n0[tt] & 1) == 0, tok + 1 < p.n_tok && t + 1 < p.t_cap);
    else put_row_i8<RT>(p, rows[i], pl, seq + sq, kv, t, on);
  }
}
// AT_ONCE rows' codes side by side
template <int R, int CT, int TT, bool I4, bool SPAN, int AT_ONCE = 1>
WSVD_DEV void project_store(const ProjectParams& p, const v16f (&acc)[CT][TT], int ct0, int row0, int seq, const int (&n0)[TT]) {
#pragma unroll
  for (int h = 0; h < CT / (R / 32); h++)
#pragma unroll
    for (int tt = 0; tt < TT; tt += AT_ONCE) project_store_tiles<R, CT, TT, I4, SPAN, AT_ONCE>(p, acc, h, tt, ct0, row0, seq, n0);
}

template <int R, int CT, int TT, int WC, bool I4 = false, int ST = 3>
__global__ __launch_bounds__(256) void k_prefill_project(ProjectParams p) {
  constexpr int RT = R / 32;
  static_assert(CT % RT == 0, "a head's channels stay in one wave");
  const int lane = threadIdx.x & 63, wave = threadIdx.x >> 6, n = lane & 31, g2 = lane >> 5;
  const int tiles_plane = p.Hkv * RT, tiles = 2 * tiles_plane;
  const int ct0 = (blockIdx.x * WC + wave % WC) * CT;                   // first channel tile of this wave
  const int tb = blockIdx.y * (4 / WC) + wave / WC;                     // its group of TT token tiles
  if (ct0 >= tiles || tb * 32 * TT >= p.n_tok) return;
  const int seq = p.seq0 + blockIdx.z;
  int n0[TT];
#pragma unroll
  for (int tt = 0; tt < TT; tt++) n0[tt] = row_length<false>(p, seq, 0);
  const int n_steps = p.E >> 4;
  const uint16_t* ap[CT];
#pragma unroll
  for (int c = 0; c < CT; c++) {
    const int ct = min(ct0 + c, tiles - 1);
    ap[c] = p.A[ct / tiles_plane] + ((size_t)(ct % tiles_plane) * n_steps * 64 + lane) * 8;
  }
  const uint16_t* xp[TT];
#pragma unroll
  for (int tt = 0; tt < TT; tt++) {
    const int tok = min((tb * TT + tt) * 32 + n, p.n_tok - 1);
    xp[tt] = p.x + ((size_t)blockIdx.z * p.n_tok + tok) * p.E + 8 * g2;
  }
  v16f acc[CT][TT];
#pragma unroll
  for (int c = 0; c < CT; c++)
#pragma unroll
    for (int tt = 0; tt < TT; tt++)
#pragma unroll
      for (int v = 0; v < 16; v++) acc[c][tt][v] = 0.f;
  v8bf16 fa[ST][CT], fb[ST][TT];
  auto fetch = [&](int st, int ks) {
    ks = min(ks, n_steps - 1);
#pragma unroll
    for (int c = 0; c < CT; c++) fa[st][c] = *(const v8bf16*)(ap[c] + (size_t)ks * 512);
#pragma unroll
    for (int tt = 0; tt < TT; tt++) fb[st][tt] = *(const v8bf16*)(xp[tt] + 16 * ks);
  };
#pragma unroll
  for (int u = 0; u < ST - 1; u++) fetch(u, u);
  for (int ks0 = 0; ks0 < n_steps; ks0 += ST) {
#pragma unroll
    for (int u = 0; u < ST; u++) {
      fetch((u + ST - 1) % ST, ks0 + u + ST - 1);
      if (ks0 + u < n_steps) {
#pragma unroll
        for (int c = 0; c < CT; c++)
#pragma unroll
          for (int tt = 0; tt < TT; tt++) acc[c][tt] = mfma_bf16(fa[u][c], fb[u][tt], acc[c][tt]);
      }
    }
  }
  project_store<R, CT, TT, I4, false>(p, acc, ct0, tb * TT * 32, seq, n0);
}

// The same projection with both operands staged through LDS: a workgroup of 8 waves (2 x 4, each 4 x 2 tiles) owns
// 256 channels x 256 tokens.  Per chunk of 64 model dims 32 KiB of the factor image (already in operand order) and 256 whole
// 128-byte lines of hidden states go from memory straight to LDS, two chunks of A and three of x deep (all 160 KiB), one barrier
// per chunk, no register and no LDS write instruction in between.  E must be a multiple of 64.
// Bound: matrix cores and LDS reads (24 KiB per wave and chunk, 1536 cycles of a CU's 128 bytes a clock beside 2048 of
// products), at the clock the power leaves; then the store, in which the matrix cores idle.  32 heads of rank 32, 16 x 2048
// tokens, d_model 4096 / 512 / 64: 449 / 103 / 49 us; through registers, two stages and rows padded to 144 bytes 518 / 117 / 60;
// this copy with 4 waves of 4 x 4 tiles (a third less to read, one wave per SIMD for the store) 462 / 128 / 78.
typedef uint32_t v4u __attribute__((ext_vector_type(4)));
constexpr int kProjKC = 64, kProjXRow = 144;
constexpr int kProjABytes = 8 * 4 * 1024, kProjXBytes = 256 * 128, kProjLds = 2 * kProjABytes + 3 * kProjXBytes;

// Workgroup -> (channel group, token group).  Consecutive workgroup ids land on different XCDs (8 of them, each with
// its own L2).  Token-affine: XCD i takes the token groups = i (mod 8), so a line of hidden states is fetched by one XCD
// only and every XCD walks through all factors.  Otherwise the channel groups go round: with a number of them that shares
// factors with 8, an XCD sees the same few channel groups all the time and all tokens.  The 256 x 256 tiles are
// token-affine where the number of token groups allows it (either way within 2 %).  The smaller tiles keep the factors with
// an XCD, unless their groups are odd in number (each XCD would see all of them anyway) or all factors fit an L2 and the
// tokens are the larger operand.  us per call, factors / tokens kept, 32 kv heads of rank 32, d_model 4096 (16.8 MB of
// factors), 128 x 32 tiles: 16 x 3 tokens 21 / 27, 64 x 16 61 / 79, 2 x 2048 129 / 164; rank 64: 16 x 16 35 / 46, 64 x 4
// 95 / 154, 8 x 1024 401 / 905; 18 heads of rank 64 (9 groups): 16 x 64 66 / 57; 16 heads of rank 32, d_model 2048 (4.2 MB):
// 16 x 16 13.6 / 16.2, 8 x 1024 75 / 70; 8 heads of rank 64, d_model 4096 (8.4 MB): 16 x 16 32 / 35, 8 x 700 85 / 80.
WSVD_DEV void project_groups(const ProjectParams& p, int& cg, int& tg) {
  const int L = blockIdx.x;
  if (p.token_affine) { const int sl = L >> 3; cg = sl % p.n_cg; tg = (sl / p.n_cg) * 8 + (L & 7); }
  else { cg = L % p.n_cg; tg = L / p.n_cg; }
}

constexpr int kProjWaves = 8;
template <int R, bool I4, bool SPAN>
__global__ __launch_bounds__(64 * kProjWaves) void k_prefill_project_lds(ProjectParams p) {
  extern __shared__ __align__(16) uint8_t proj_lds[];                   // two stages of A, three of x
  constexpr int RT = R / 32, WAVES = kProjWaves, CT = 4, TT = 16 / WAVES, NS = kProjKC / 16;     // 2 x (WAVES / 2) waves, each 4 x TT tiles
  constexpr int NA = 8 / WAVES, NX = 32 / WAVES;                        // channel tiles, groups of 8 rows a wave copies
  const int lane = threadIdx.x & 63, n = lane & 31, g2 = lane >> 5;
  const int wave = __builtin_amdgcn_readfirstlane(threadIdx.x >> 6), wc = wave & 1, wt = wave >> 1;
  const int tiles_plane = p.Hkv * RT, tiles = 2 * tiles_plane;
  int cg, tg;
  project_groups(p, cg, tg);
  const int sq = tg / p.tg_seq, by = tg % p.tg_seq;                     // set of rows, 256-row group in it
  const int seq = p.seq0 + sq;                                          // (its first sequence)
  const int ct0 = (cg * 2 + wc) * CT, row0 = by * 256 + wt * 32 * TT;
  int n0[TT];
#pragma unroll
  for (int tt = 0; tt < TT; tt++) n0[tt] = row_length<SPAN>(p, seq, row0 + 32 * tt + n);
  const int n_steps = p.E >> 4, n_chunks = p.E / kProjKC;
  // What this wave copies per chunk, 1 KiB per instruction: two channel tiles of A, which are in operand order, and 64 token
  // rows, 8 of them (whole 128-byte lines) at a time.  LDS takes what the lanes bring in lane order, so a row's 16-byte
  // pieces are swapped on the way in: piece s of row r goes to place s ^ (r & 7), and 8 neighbouring rows' pieces of one
  // column lie in 8 different places, without padding.  (Rows r and r + 8 meet: two rows of 128 bytes share the 256 bytes of all banks.
  // SQ_LDS_BANK_CONFLICT counts four cycles per read, 65 k of a CU's 900 k at 16 x 2048 tokens.)
  const uint8_t* asrc[NA];
#pragma unroll
  for (int j = 0; j < NA; j++) {
    const int ct = min(cg * 8 + NA * wave + j, tiles - 1);
    asrc[j] = (const uint8_t*)p.A[ct / tiles_plane] + (size_t)(ct % tiles_plane) * n_steps * 1024;
  }
  const uint8_t* const xbase = (const uint8_t*)p.x + (size_t)sq * p.n_tok * p.E * 2;
  const uint32_t lane16 = lane * 16;
  uint32_t xoff[NX];
#pragma unroll
  for (int j = 0; j < NX; j++) {
    const int row = by * 256 + 8 * NX * wave + 8 * j + (lane >> 3);         // the launcher keeps rows * E * 2 below 2^31
    xoff[j] = (uint32_t)min(row, p.rows - 1) * (uint32_t)(p.E * 2) + (((lane & 7) ^ (lane >> 3)) * 16);
  }
  const uint32_t lds0 = __builtin_amdgcn_readfirstlane(lds_address(proj_lds));
  // (past the end: the last chunk again, into a stage that is not read any more)
  auto copy_a = [&](int j, int ks, int c) {
    lds_copy16(lds0 + (c & 1) * kProjABytes + (NA * wave + j) * 4096 + ks * 1024, asrc[j] + (size_t)min(c, n_chunks - 1) * 4096 + ks * 1024, lane16);
  };
  auto copy_x = [&](int j, int c, int st) {
    lds_copy16(lds0 + 2 * kProjABytes + st * kProjXBytes + (8 * NX * wave + 8 * j) * 128, xbase + (size_t)min(c, n_chunks - 1) * (kProjKC * 2), xoff[j]);
  };
  v16f acc[CT][TT];
#pragma unroll
  for (int c = 0; c < CT; c++)
#pragma unroll
    for (int tt = 0; tt < TT; tt++)
#pragma unroll
      for (int v = 0; v < 16; v++) acc[c][tt][v] = 0.f;
  const uint8_t* const a_at = proj_lds + wc * 4 * 4096 + lane16;                             // + stage + tile * 4096 + step * 1024
  const uint8_t* const x_at = proj_lds + 2 * kProjABytes + (wt * 32 * TT + n) * 128;             // + stage + tile * 4096 + place
  const uint32_t place = ((uint32_t)g2 ^ (n & 7)) * 16;                                      // ^ step * 32
  v8bf16 fa[2][CT], fb[2][TT];
  auto read_a = [&](int b, int cc, int ks, int c) { fa[b][cc] = *(const v8bf16*)(a_at + (c & 1) * kProjABytes + cc * 4096 + ks * 1024); };
  auto read_x = [&](int b, int tt, int ks, int st) { fb[b][tt] = *(const v8bf16*)(x_at + st * kProjXBytes + tt * 4096 + (place ^ (ks * 32))); };
#pragma unroll
  for (int ks = 0; ks < NS; ks++)
#pragma unroll
    for (int j = 0; j < NA; j++) copy_a(j, ks, 0);
#pragma unroll
  for (int j = 0; j < NX; j++) copy_x(j, 0, 0);
#pragma unroll
  for (int j = 0; j < NX; j++) copy_x(j, 1, 1);
  project_hold(n0);
  lds_copy_wait_barrier<NX>();
#pragma unroll
  for (int i = 0; i < 4; i++) { read_a(0, i, 0, 0); if (i < TT) read_x(0, i, 0, 0); }
  // Per chunk four steps of 16 products.  The operands of a step are read during the step before it, those of a chunk's
  // first step during the last step of the chunk before: the chunk's only barrier stands in front of that last step, when all
  // reads of the chunk have been answered and (the wait) this wave's copies of the next chunk have arrived.  Behind the
  // barrier the stages of the chunk may be overwritten: A of the next but one and x of the next but two are asked for
  // there and in the next chunk's first step, a chunk and two chunks before they are needed.
  int st = 0;                                                           // stage of x
  for (int c = 0; c < n_chunks; c++) {
    const int st1 = st == 2 ? 0 : st + 1, st2 = st1 == 2 ? 0 : st1 + 1;
#pragma unroll
    for (int ks = 0; ks < NS; ks++) {
      const int b = ks & 1;
      if (ks == NS - 1) {
        __builtin_amdgcn_sched_barrier(0);
        lds_copy_wait_barrier<NX>();
      }
#pragma unroll
      for (int cc = 0; cc < CT; cc++) {
        __builtin_amdgcn_sched_barrier(0);
        if (ks < NS - 1) { read_a(b ^ 1, cc, ks + 1, c); if (cc < TT) read_x(b ^ 1, cc, ks + 1, st); }
        else { read_a(b ^ 1, cc, 0, c + 1); if (cc < TT) read_x(b ^ 1, cc, 0, st1); }
        __builtin_amdgcn_sched_barrier(0);
#pragma unroll
        for (int tt = 0; tt < TT; tt++) {
          acc[cc][tt] = mfma_bf16(fa[b][cc], fb[b][tt], acc[cc][tt]);
          __builtin_amdgcn_sched_barrier(0);
          if (ks == 0 && tt < NA) copy_a(tt, cc, c + 1);
          if (ks == 1 && tt < NX / 4) copy_x(NX / 4 * cc + tt, c + 2, st2);
        }
      }
    }
    st = st1;
  }
  if (ct0 >= tiles || row0 >= p.rows) return;                           // (never the first wave)
  const int seen = project_count(p);
  project_store<R, CT, TT, I4, SPAN, TT>(p, acc, ct0, row0, seq, n0);
  project_advance(p, seen);
}

// The projection with the hidden states staged through LDS and the factors straight from memory into the registers that
// feed the matrix cores (the packed image is the operand, a wave's channels are its own, so LDS would only cost it a write
// and a read).  A workgroup owns 32 CT WC channels x 32 TT rows; its waves are KS groups of WC (wave w of a group: the CT
// channel tiles from CT (WC cg + w) on, all of the workgroup's rows).  Group g takes the chunks g, g + KS, .. of 64 model dims
// through two LDS stages of its own, DEPTH chunks on their way in registers, one barrier per round; the groups' sums meet in
// LDS.  For problems that do not fill the chip with 256 x 256 tiles.  What bounds it is what a CU takes in, 64 bytes a clock
// (126 B/ns measured out of L2 on few CUs, 95 to 105 on all): (channels + rows) x d_model x 2 bytes per workgroup, 128 x 32
// at 125 B/ns, 128 x 64 at 72 with all CUs busy.  Hence as few bytes as the number of workgroups allows (project_shape_rule),
// and the contraction split inside the workgroup where its tile is too small to keep 8 waves busy otherwise.
template <int R, int CT, int TT, int WC, int KS, int DEPTH, bool I4, bool SPAN>
__global__ __launch_bounds__(64 * WC * KS) void k_prefill_project_direct(ProjectParams p) {
  constexpr int RT = R / 32;
  static_assert(CT % RT == 0, "a head's channels stay in one wave");
  static_assert(DEPTH % 2 == 0, "LDS stage and register set follow from the position in the unrolled loop");
  static_assert((4 * TT) % WC == 0, "a group's threads copy whole rows");
  constexpr int NX = 4 * TT / WC, NS = kProjKC / 16;                    // 16-byte pieces of x per thread and chunk; steps
  constexpr int STAGE = 32 * TT * kProjXRow;
  extern __shared__ __align__(16) uint8_t proj_lds[];
  const int lane = threadIdx.x & 63, n = lane & 31, g2 = lane >> 5;
  const int wave = __builtin_amdgcn_readfirstlane(threadIdx.x >> 6), wc = wave % WC, kg = wave / WC;
  const int gt = wc * 64 + lane;                                        // thread of its group
  uint8_t* const lds = proj_lds + kg * 2 * STAGE;
  const int tiles_plane = p.Hkv * RT, tiles = 2 * tiles_plane;
  int cg, tg;
  project_groups(p, cg, tg);
  const int sq = tg / p.tg_seq, by = tg % p.tg_seq;
  const int seq = p.seq0 + sq;
  const int n_steps = p.E >> 4, n_chunks = p.E / kProjKC, n_iter = (n_chunks + KS - 1) / KS;
  const int ct0 = (cg * WC + wc) * CT;                                  // first channel tile of this wave
  const uint8_t* asrc[CT];
#pragma unroll
  for (int c = 0; c < CT; c++) {
    const int ct = min(ct0 + c, tiles - 1);
    asrc[c] = (const uint8_t*)p.A[ct / tiles_plane] + (size_t)(ct % tiles_plane) * n_steps * 1024;
  }
  const uint8_t* xbase = (const uint8_t*)p.x + (size_t)sq * p.n_tok * p.E * 2;
  uint32_t xoff[NX];
#pragma unroll
  for (int j = 0; j < NX; j++)                                          // (the launcher keeps rows * E * 2 below 2^31)
    xoff[j] = (uint32_t)min(by * 32 * TT + (gt >> 3) + 8 * WC * j, p.rows - 1) * (uint32_t)(p.E * 2) + (gt & 7) * 16;
  const int xdst = (gt >> 3) * kProjXRow + (gt & 7) * 16;               // + 8 WC j rows
  const uint32_t aoff = lane * 16;
  v8bf16 ra[DEPTH][CT][NS];
  v4u rx[DEPTH][NX];
  auto chunk = [&](int it) { return min(it * KS + kg, n_chunks - 1); }; // (past the end: the last chunk again, not used)
  auto fetch_a = [&](int b, int it) {
    const int c = chunk(it);
#pragma unroll
    for (int cc = 0; cc < CT; cc++)
#pragma unroll
      for (int ks = 0; ks < NS; ks++) ra[b][cc][ks] = *(const v8bf16*)((asrc[cc] + (size_t)c * 4096 + ks * 1024) + aoff);
  };
  auto fetch_x = [&](int b, int it) {
    const int c = chunk(it);
#pragma unroll
    for (int j = 0; j < NX; j++) rx[b][j] = *(const v4u*)((xbase + (size_t)c * (kProjKC * 2)) + xoff[j]);
  };
  auto commit = [&](int b, int st) {
#pragma unroll
    for (int j = 0; j < NX; j++) *(v4u*)(lds + st * STAGE + 8 * WC * j * kProjXRow + xdst) = rx[b][j];
  };
  v16f acc[CT][TT];
#pragma unroll
  for (int c = 0; c < CT; c++)
#pragma unroll
    for (int tt = 0; tt < TT; tt++)
#pragma unroll
      for (int v = 0; v < 16; v++) acc[c][tt][v] = 0.f;
#pragma unroll
  for (int u = 0; u < DEPTH; u++) { fetch_x(u, u); fetch_a(u, u); }
  commit(0, 0);
  fetch_x(0, DEPTH);
  __syncthreads();
  const int x_off = n * kProjXRow + g2 * 16;
  // round it of the group's chunks sits in LDS stage it & 1 and in factor set it % DEPTH; set (it + 1) % DEPTH of the hidden
  // states holds round it + 1
  auto round = [&](int u, int it, bool mine) {                          // (u = it % DEPTH, a constant after unrolling)
    commit((u + 1) % DEPTH, (u + 1) & 1);
    fetch_x((u + 1) % DEPTH, it + 1 + DEPTH);
    const uint8_t* base = lds + (u & 1) * STAGE + x_off;
    if (mine) {
#pragma unroll
      for (int ks = 0; ks < NS; ks++) {
        v8bf16 fb[TT];
#pragma unroll
        for (int tt = 0; tt < TT; tt++) fb[tt] = *(const v8bf16*)(base + tt * 32 * kProjXRow + ks * 32);
#pragma unroll
        for (int cc = 0; cc < CT; cc++)
#pragma unroll
          for (int tt = 0; tt < TT; tt++) acc[cc][tt] = mfma_bf16(ra[u][cc][ks], fb[tt], acc[cc][tt]);
      }
    }
    fetch_a(u, it + DEPTH);
    __syncthreads();
  };
  // The loop takes DEPTH rounds at a time and has no branch inside: with a round that could be skipped, the compiler has to
  // assume that only the last one's requests are in flight and drains all of them once per DEPTH rounds, which doubled the time.
  const int n_main = n_chunks / KS / DEPTH * DEPTH;
  for (int it = 0; it < n_main; it += DEPTH) {
#pragma unroll
    for (int u = 0; u < DEPTH; u++) round(u, it + u, true);
  }
  for (int it = n_main; it < n_iter; it += DEPTH) {
#pragma unroll
    for (int u = 0; u < DEPTH; u++)
      if (it + u < n_iter) round(u, it + u, (it + u) * KS + kg < n_chunks);
  }
  int n0[TT];                                                           // (asked for here: no registers during the products)
#pragma unroll
  for (int tt = 0; tt < TT; tt++) n0[tt] = row_length<SPAN>(p, seq, (by * TT + tt) * 32 + (lane_number() & 31));
  // (counted behind the store where no register is left to hold the answer)
  constexpr bool LATE = R == 64 && CT * TT >= 8;
  int seen = -1;
  if constexpr (!LATE) project_hold(n0);
  if constexpr (KS == 1) {
    __syncthreads();
    if constexpr (!LATE) seen = project_count(p);
    if (ct0 >= tiles) return;                                           // (never the first wave)
    project_store<R, CT, TT, I4, SPAN>(p, acc, ct0, by * 32 * TT, seq, n0);
  } else {
    // the groups' sums meet in LDS: unit u (the channels of a head x 32 rows) is added up in group order and stored by group
    // u % KS, from the pieces the other groups leave there
    constexpr int NU = CT / RT * TT;
    float* const mine = (float*)proj_lds + lane_number();
    auto piece = [&](int u, int g) { return ((u * (KS - 1) + (g > u % KS ? g - 1 : g)) * WC + wc) * (RT * 1024); };
#pragma unroll
    for (int u = 0; u < NU; u++) {
      if (u % KS == kg) continue;
      const int at = piece(u, kg);
#pragma unroll
      for (int rt = 0; rt < RT; rt++)
#pragma unroll
        for (int v = 0; v < 16; v++) mine[at + (rt * 16 + v) * 64] = acc[u / TT * RT + rt][u % TT][v];
    }
    __syncthreads();
    if constexpr (!LATE) seen = project_count(p);
    if (ct0 >= tiles) return;
#pragma unroll
    for (int u = 0; u < NU; u++) {
      if (u % KS != kg) continue;
#pragma unroll
      for (int rt = 0; rt < RT; rt++)
#pragma unroll
        for (int v = 0; v < 16; v++) {
          float sum = 0.f;
#pragma unroll
          for (int g = 0; g < KS; g++) {
            const float x = g == u % KS ? acc[u / TT * RT + rt][u % TT][v] : mine[piece(u, g) + (rt * 16 + v) * 64];
            sum = g ? sum + x : x;
          }
          acc[u / TT * RT + rt][u % TT][v] = sum;
        }
      project_store_tiles<R, CT, TT, I4, SPAN, 1>(p, acc, u / TT, u % TT, ct0, by * 32 * TT, seq, n0);
    }
  }
  if constexpr (LATE) {
    __syncthreads();                                                    // (every wave has used its lengths)
    seen = project_count(p);
  }
  project_advance(p, seen);
}

// the same behind k_prefill_project, one thread per sequence
__global__ void k_prefill_bump(int* seq_lens, int seq0, int n_seq, int n_tok, int t_cap, int* err_word, int even_only) {
  const int i = blockIdx.x * blockDim.x + threadIdx.x;
  if (i < n_seq) project_bump(seq_lens, seq0 + i, n_tok, t_cap, err_word, even_only);
}

template <int R, int CT, int TT, int WC, bool I4 = false>
void launch_project(const ProjectParams& p, int n_seq, hipStream_t s) {
  const int tiles = 2 * p.Hkv * (R / 32), tok_wg = 32 * TT * (4 / WC);
  dim3 grid((unsigned)((tiles + WC * CT - 1) / (WC * CT)), (unsigned)((p.n_tok + tok_wg - 1) / tok_wg), (unsigned)n_seq);
  hipLaunchKernelGGL((k_prefill_project<R, CT, TT, WC, I4>), grid, dim3(256), 0, s, p);
}

void project_grid(ProjectParams& p, int n_seq, int ch_wg, int tok_wg, int R, bool i4) {
  // Tiles across sequences where that saves a round of workgroups (a last tile of few rows is cheap: 16 x 260 tokens, three
  // rounds of 256 x 64 either way, 105 us in 640 workgroups and 110 in 520; 64 x 4 tokens 53 and 16) and the rows' offsets fit
  // 32 bits; int4 stores pair the rows of neighbouring lanes, so there a sequence has to begin in an even lane.
  p.n_cg = (2 * p.Hkv * R + ch_wg - 1) / ch_wg;
  const long long own = (long long)((p.n_tok + tok_wg - 1) / tok_wg) * n_seq, all = ((long long)n_seq * p.n_tok + tok_wg - 1) / tok_wg;
  const bool span = (all * p.n_cg + 255) / 256 < (own * p.n_cg + 255) / 256 && (long long)n_seq * p.n_tok * p.E * 2 < (1LL << 31) &&
                    (!i4 || p.n_tok % 2 == 0);
  p.rows = span ? n_seq * p.n_tok : p.n_tok;
  p.n_tg = (int)(span ? all : own);
  p.tg_seq = span ? p.n_tg : (int)(own / n_seq);
  p.token_affine = p.n_tg % 8 == 0;
}

template <int R, int CT, int TT, int WC, int KS, int DEPTH, bool I4, bool SPAN>
hipError_t launch_project_direct_span(const ProjectParams& p, hipStream_t s) {
  constexpr int RT = R / 32, STAGES = KS * 2 * 32 * TT * kProjXRow, PIECES = CT / RT * TT * (KS - 1) * WC * RT * 4096;
  constexpr int LDS = STAGES > PIECES ? STAGES : PIECES;
  if constexpr (LDS > 65536) {
    static LdsLimit limit;
    hipError_t e = wsvd_raise_lds(limit, (const void*)k_prefill_project_direct<R, CT, TT, WC, KS, DEPTH, I4, SPAN>, LDS);
    if (e != hipSuccess) return e;
  }
  hipLaunchKernelGGL((k_prefill_project_direct<R, CT, TT, WC, KS, DEPTH, I4, SPAN>), dim3((unsigned)(p.n_cg * p.n_tg)), dim3(64 * WC * KS), LDS, s, p);
  return hipGetLastError();
}
// (tiles that stay inside a sequence keep its plane's address in scalar registers: 2 to 3 % of short calls, 1.5 % of 16 x 2048
// tokens in 256 x 256 tiles)
template <int R, int CT, int TT, int WC, int KS, int DEPTH, bool I4 = false>
hipError_t launch_project_direct(ProjectParams p, int n_seq, hipStream_t s) {
  project_grid(p, n_seq, 32 * WC * CT, 32 * TT, R, I4);
  // (which operand stays with an XCD: see project_groups)
  const long long ch = 2LL * p.Hkv * R;
  const bool l2_holds_factors = ch * p.E * 2 <= (9LL << 20);
  if (p.n_cg % 2 == 0 && !(l2_holds_factors && (long long)n_seq * p.n_tok >= ch)) p.token_affine = false;
  return p.rows == p.n_tok ? launch_project_direct_span<R, CT, TT, WC, KS, DEPTH, I4, false>(p, s) :
                             launch_project_direct_span<R, CT, TT, WC, KS, DEPTH, I4, true>(p, s);
}

template <int R, bool I4, bool SPAN>
hipError_t launch_project_lds_span(const ProjectParams& p, hipStream_t s) {
  static LdsLimit limit;
  const size_t lds = kProjLds;
  hipError_t e = wsvd_raise_lds(limit, (const void*)k_prefill_project_lds<R, I4, SPAN>, (int)lds);
  if (e != hipSuccess) return e;
  hipLaunchKernelGGL((k_prefill_project_lds<R, I4, SPAN>), dim3((unsigned)(p.n_cg * p.n_tg)), dim3(64 * kProjWaves), lds, s, p);
  return hipGetLastError();
}
template <int R, bool I4 = false>
hipError_t launch_project_lds(ProjectParams p, int n_seq, hipStream_t s) {
  project_grid(p, n_seq, 256, 256, R, I4);
  return p.rows == p.n_tok ? launch_project_lds_span<R, I4, false>(p, s) : launch_project_lds_span<R, I4, true>(p, s);
}

// The tile size.  256 workgroups (one per CU) run side by side.  A round of them costs chain * d_model / 4096 us for the
// contraction; what grows with the work that a round holds, the store of the rows and what the memory system adds, counts full
// rounds once and the last one by the square of the share of the CUs that it keeps busy, because a CU has the next workgroup
// beside it; `fixed` (first requests, sums, last store) shows once.  The shape that costs least.  Smaller tiles read the operands
// more often (see k_prefill_project_direct), larger ones leave CUs idle.  The constants are fitted to 840 sizes (1 to 40 heads of
// rank 32 or 64, d_model 64 to 8192, 2 to 40000 tokens): the choice is 0.7 % slower than the best of the shapes on average, 0.3
// from d_model 512 on (0.4 over 170 sizes with the operands out of memory).  Those of 22, 25 and 2 are fitted again to 136 sizes of
// 512 to 40000 tokens (choice 0.5 % slower than the best on average; 2.5 with the constants of the 256 x 256 tiles before they were
// copied straight to LDS: 6 x 1000 tokens 117 us then, 96 now).  us per call with the update of the lengths and the clearing before
// it (all but the last row measured with the update as a launch of its own, about 1 us), 32 kv heads of rank
// 32 / 64, d_model 4096; the last column 28 x 385 tokens at d_model 192, where the store is most of the time:
//                   1 x 200   16 x 32   1 x 400   3 x 333   4 x 500  16 x 130  2 x 2048  8 x 1024    64 x 4    28 x 385
//    5:  64 x  32     16/23     25/42     24/40     41/77    71/147    78/156   141/288   267/553     17/24      79/189
//   11: 128 x  32     20/22     22/36     20/34     35/63    62/119    73/134   119/229   230/456     20/23      48/133
//   12: 128 x  64     25/30     27/31     26/31     31/49     53/89    71/106   101/168   192/342     26/31      64/84
//   22: 256 x  64     42/41     41/43     42/42     43/47     47/78    72/111    84/149   158/304     44/42      46/69
//   25: 256 x 128     54/55     53/59     56/55     57/56     57/69    65/122    74/135   141/267     56/57      47/79
//    2: 256 x 256      78/75     81/99     77/76     80/80     80/85    82/107    82/118   121/233     78/77     32/60
// 13, 256 x 32, is there for rank 64: it reads the hidden states half as often as 11 and is the best where the contraction is
// short (30 x 46 tokens of 8 heads, d_model 192: 10.0 us, the others 10.9 and more); its chain is priced for that, at larger
// d_model 12 and 22 are as fast.
// A shape that sums the contraction in one chain has to be 2 % cheaper (256 x 256: 6 %) than one that halves it over wave groups, whose
// sums are nearer to the exact ones (scales of 10 x 1178 tokens, d_model 512, against 64 bits: 4.2e-6 and 3.3e-6).
struct ProjectShape { int code, ch, tok; bool halves[2]; float fixed[2], store[2], chain, busy; };   // pairs: rank 32, 64
constexpr ProjectShape kProjectShapes[] = {
    {5, 64, 32, {true, true}, {0.9f, 1.8f}, {0.9f, 1.2f}, 7.5f, 0.3f},
    {11, 128, 32, {false, true}, {0.9f, 2.3f}, {1.05f, 1.7f}, 11.2f, 1.5f},
    {12, 128, 64, {true, true}, {2.3f, 2.6f}, {3.4f, 1.9f}, 17.5f, 1.7f},
    {13, 256, 32, {false, false}, {-1.f, 1.5f}, {0.f, 1.9f}, 26.f, 0.f},
    {22, 256, 64, {false, false}, {3.9f, 2.5f}, {2.7f, 2.8f}, 31.8f, 1.6f},
    {25, 256, 128, {true, true}, {5.0f, 0.6f}, {6.5f, 6.9f}, 47.7f, 9.8f},
    {2, 256, 256, {false, false}, {6.5f, 4.5f}, {8.0f, 7.7f}, 64.7f, 33.3f}};
int project_shape_rule(const ProjectParams& p, int n_seq, int R, bool i4) {
  int best[2] = {0, 0};                                                 // of the shapes that sum in one chain, of those that halve it
  float least[2] = {INFINITY, INFINITY};
  for (const ProjectShape& k : kProjectShapes) {
    const int r = R == 64, halves = k.halves[r];
    if (k.fixed[r] < 0.f) continue;                                     // not there at this rank
    ProjectParams g = p;
    project_grid(g, n_seq, k.ch, k.tok, R, i4);
    const float wgs = (float)g.n_cg * (float)g.n_tg, rounds = ceilf(wgs / 256.f), load = wgs / 256.f - (rounds - 1.f);
    const float held = rounds - 1.f + load * load;
    const float us = 6.f + k.fixed[r] + k.store[r] * held + (rounds * k.chain + held * k.busy) * (float)p.E / 4096.f;
    if (us < least[halves]) { best[halves] = k.code; least[halves] = us; }
  }
  return least[0] * (best[0] == 2 ? 1.06f : 1.02f) < least[1] ? best[0] : best[1];
}

}  // namespace


hipError_t wsvd_launch_prefill_project(const wsvd_ctx* ctx, const wsvd_layer_desc& d, const void* x, int n_tok, int seq,
                                       const void* A_K, const void* A_V, const wsvd_cache& cache, hipStream_t s,
                                       const wsvd_paged_cache* paged) {
  const bool i4 = d.latent_dtype == WSVD_I4 && d.rank == 32;
  if (paged && d.rank > 64) return hipErrorNotSupported;
  if ((d.latent_dtype != WSVD_I8 && !i4) || d.factor_dtype != WSVD_BF16 || d.x_dtype != WSVD_BF16) return hipErrorNotSupported;
  if (d.rank != 32 && d.rank != 64 && d.rank != 96 && d.rank != 128) return hipErrorNotSupported;
  if (d.d_model % 16 != 0 || n_tok < 1) return hipErrorInvalidValue;
  ProjectParams p;
  p.x = (const uint16_t*)x; p.A[0] = (const uint16_t*)A_K; p.A[1] = (const uint16_t*)A_V;
  p.codes[0] = (uint8_t*)cache.k_codes; p.codes[1] = (uint8_t*)cache.v_codes;
  p.meta[0] = (uint16_t*)cache.k_meta; p.meta[1] = (uint16_t*)cache.v_meta;
  p.seq_lens = cache.seq_lens; p.err_word = ctx->err_word;
  p.Hkv = d.n_kv_heads; p.E = d.d_model; p.t_cap = d.t_cap; p.n_tok = p.rows = n_tok;
  p.n_cg = p.tg_seq = p.n_tg = 0; p.token_affine = false;
  p.block_table = nullptr; p.page_rows = p.max_pages = p.n_pages = 0;
  if (paged) { p.block_table = paged->block_table; p.page_rows = paged->page_rows; p.max_pages = paged->max_pages; p.n_pages = paged->n_pages; }
  const int n_seq = seq < 0 ? d.batch : 1;
  p.seq0 = seq < 0 ? 0 : seq;
  p.readers = ctx->readers; p.n_seq = n_seq; p.even_only = i4 ? 1 : 0;
  const bool tiles_ok = d.d_model % kProjKC == 0 && (long long)n_tok * d.d_model * 2 < (1LL << 31);
  int shape = ctx->opt.project_shape;
  if (!shape) shape = project_shape_rule(p, n_seq, d.rank, i4);
  if (shape == 13 && d.rank == 32) shape = 11;
  const bool direct = shape == 5 || shape == 11 || shape == 12 || shape == 13 || shape == 22 || shape == 25;
  if (!tiles_ok || !direct) shape = tiles_ok && shape <= 2 ? 2 : 44;
  hipError_t e = hipSuccess;
  if (d.rank > 64) {
    // ranks 96 / 128: a wave owns the 3 / 4 channel tiles of one head and 1 or 4 token tiles
    const bool big = (long long)n_seq * n_tok * d.n_kv_heads * d.rank >= (1LL << 22);
    if (d.rank == 96) { if (big) launch_project<96, 3, 4, 4>(p, n_seq, s); else launch_project<96, 3, 1, 4>(p, n_seq, s); }
    else { if (big) launch_project<128, 4, 4, 4>(p, n_seq, s); else launch_project<128, 4, 1, 4>(p, n_seq, s); }
  } else if (shape == 5) {
    if (i4) e = launch_project_direct<32, 1, 1, 2, 2, 4, true>(p, n_seq, s);
    else if (d.rank == 32) e = launch_project_direct<32, 1, 1, 2, 2, 4>(p, n_seq, s);
    else e = launch_project_direct<64, 2, 1, 1, 2, 4>(p, n_seq, s);
  } else if (shape == 11) {
    if (i4) e = launch_project_direct<32, 1, 1, 4, 1, 4, true>(p, n_seq, s);
    else if (d.rank == 32) e = launch_project_direct<32, 1, 1, 4, 1, 4>(p, n_seq, s);
    else e = launch_project_direct<64, 2, 1, 2, 2, 4>(p, n_seq, s);
  } else if (shape == 12) {
    if (i4) e = launch_project_direct<32, 1, 2, 4, 2, 4, true>(p, n_seq, s);
    else if (d.rank == 32) e = launch_project_direct<32, 1, 2, 4, 2, 4>(p, n_seq, s);
    else e = launch_project_direct<64, 2, 2, 2, 2, 2>(p, n_seq, s);
  } else if (shape == 13) {
    e = launch_project_direct<64, 2, 1, 4, 1, 4>(p, n_seq, s);
  } else if (shape == 22) {
    if (i4) e = launch_project_direct<32, 2, 2, 4, 1, 4, true>(p, n_seq, s);
    else if (d.rank == 32) e = launch_project_direct<32, 2, 2, 4, 1, 4>(p, n_seq, s);
    else e = launch_project_direct<64, 2, 2, 4, 1, 4>(p, n_seq, s);
  } else if (shape == 25) {
    if (i4) e = launch_project_direct<32, 2, 4, 4, 2, 2, true>(p, n_seq, s);
    else if (d.rank == 32) e = launch_project_direct<32, 2, 4, 4, 2, 2>(p, n_seq, s);
    else e = launch_project_direct<64, 2, 4, 4, 2, 2>(p, n_seq, s);
  } else if (shape == 2) {
    if (i4) e = launch_project_lds<32, true>(p, n_seq, s);
    else if (d.rank == 32) e = launch_project_lds<32>(p, n_seq, s);
    else e = launch_project_lds<64>(p, n_seq, s);
  } else if (i4) launch_project<32, 4, 4, 4, true>(p, n_seq, s);
  else if (d.rank == 32) launch_project<32, 4, 4, 4>(p, n_seq, s);
  else launch_project<64, 4, 4, 4>(p, n_seq, s);
  if (e == hipSuccess) e = hipGetLastError();
  if (e != hipSuccess || (d.rank <= 64 && shape != 44)) return e;       // (the tile kernels have advanced the lengths)
  hipLaunchKernelGGL(k_prefill_bump, dim3((n_seq + 63) / 64), dim3(64), 0, s, cache.seq_lens, p.seq0, n_seq, n_tok, d.t_cap, ctx->err_word, i4 ? 1 : 0);
  return hipGetLastError();
}
