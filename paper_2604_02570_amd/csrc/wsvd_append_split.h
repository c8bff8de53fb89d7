// The projection of the new tokens, c = x A, as the append kernels and the decode step's launches run it: the vector-ALU
// form and the matrix-core form with helper workgroups.
#pragma once
#include "wsvd_append_body.h"

// What becomes of a workgroup's sums.  kNoDefer: this launch finishes the rows.  kDeferSlices, kDeferShares: plain stores for
// the attention launch that follows.  kPushShares: {value, tag} words for attention workgroups of the same launch, which wait
// for them, and which advance the lengths; kPushSlices: kDeferSlices that way.
enum { kNoDefer = 0, kDeferSlices = 1, kDeferShares = 2, kPushShares = 3, kPushSlices = 4 };
constexpr bool defer_pushes(int defer) { return defer == kPushShares || defer == kPushSlices; }
constexpr bool defer_slices(int defer) { return defer == kDeferSlices || defer == kPushSlices; }
constexpr uint32_t kLLTag = 0x4C4C5701u;      // marks a pushed word as written by the running launch's helper
WSVD_DEV unsigned long long ll_word(float v) { return ((unsigned long long)kLLTag << 32) | (unsigned long long)__float_as_uint(v); }
template <int DEFER>
WSVD_DEV void append_defer_out(const AppendParams& p, size_t i, float v) {
  if constexpr (defer_pushes(DEFER)) __hip_atomic_store(p.defer_words + i, ll_word(v), __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT);
  else p.defer_out[i] = v;
}

// The decode step's projection launch: sequence b's length moves on now, its row is still to be written.  A full sequence
// is reported and left alone.
WSVD_DEV void append_defer_bump(const AppendParams& p, int b, int n) {
  const bool ok = n >= 0 && n < p.t_cap;
  if (ok) p.seq_lens[b] = n + 1;
  else atomicExch(p.err_word, (int)WSVD_E_CAPACITY);
  p.pending[b] = ok ? 1 : 0;
}

// ---------------------------------------------------------------- vector-ALU path (any dtype)
// DEFER (the decode step's projection launch): the slices' partial sums are left in p.defer_out [slice][plane][B][Hkv * R]
// for the attention launch that follows, which sums them in slice order, rounds and stores the rows; workgroup 0 advances
// the lengths and marks the rows as pending.  No ticket, no read-back: 9.8 -> 6.3 us for one sequence of 8 heads, rank 16,
// d_model 512, where the ticket and the read-back were most of the launch; staging one sequence instead of eight: 5.2 us.
// BB: sequences per pass (1 for a single sequence: an eighth of the staging and of the products).
template <int R, int FESZ, int DEFER, int BB, class Params = AppendParams>
WSVD_DEV void append_valu_body(Params p, int wg) {
  constexpr int EL = 256 / R;                 // threads along d_model per latent channel
  constexpr int NA = kAppendMaxESL / EL;      // factor elements per thread
  __shared__ __attribute__((aligned(16))) float xs[kAppendMaxESL][BB];
  __shared__ float red[EL][BB][R];
  __shared__ float crow[64][R + 1];
  __shared__ int flag_sh;
  __shared__ int n_sh[kAppendMaxB];

  if constexpr (!DEFER) append_read_lens(p, n_sh);
  int s, kv, pl;
  append_coords(p, wg, s, kv, pl);
  const int tid = threadIdx.x, j = tid % R, el = tid / R;
  const int e0 = s * p.ESL;
  float* part = p.partials + ((((size_t)pl * p.Hkv + kv) * p.ES + s) * p.B) * R;

  // this thread's slice of channel j: read once (all loads in flight together), reused for every sequence
  float a[NA];
#pragma unroll
  for (int i = 0; i < NA; i++) {
    const int e = min(el + i * EL, p.ESL - 1);
    const size_t idx = a_packed_offset(kv, j, e0 + e, R, p.E);
    a[i] = FESZ == 4 ? ((const float*)p.A[pl])[idx] : bf16_to_f32(((const uint16_t*)p.A[pl])[idx]);
  }

  for (int b0 = 0; b0 < p.B; b0 += BB) {
    const int nb = min(BB, p.B - b0);
    if (b0 > 0) __syncthreads();
    for (int i = tid; i < BB * p.ESL; i += 256) {
      const int bb = BB == 1 ? 0 : i / p.ESL, e = BB == 1 ? i : i % p.ESL;
      xs[e][bb] = bb < nb ? load_x(p, b0 + bb, e0 + e) : 0.f;
    }
    __syncthreads();
    float acc[BB];
#pragma unroll
    for (int bb = 0; bb < BB; bb++) acc[bb] = 0.f;
#pragma unroll
    for (int i = 0; i < NA; i++) {
      const int e = el + i * EL;
      if (e < p.ESL) {
        if constexpr (BB == 1) {
          acc[0] = fmaf(xs[e][0], a[i], acc[0]);
        } else {
          const v4f x0 = *(const v4f*)&xs[e][0], x1 = *(const v4f*)&xs[e][4];
#pragma unroll
          for (int bb = 0; bb < 4; bb++) { acc[bb] = fmaf(x0[bb], a[i], acc[bb]); acc[4 + bb] = fmaf(x1[bb], a[i], acc[4 + bb]); }
        }
      }
    }
#pragma unroll
    for (int bb = 0; bb < BB; bb++) red[el][bb][j] = acc[bb];
    __syncthreads();
    for (int i = tid; i < nb * R; i += 256) {
      const int bb = i / R, jj = i % R;
      float sum = 0.f;
#pragma unroll
      for (int k = 0; k < EL; k++) sum += red[k][bb][jj];
      if constexpr (DEFER) append_defer_out<DEFER>(p, (((size_t)s * 2 + pl) * p.B + b0 + bb) * ((size_t)p.Hkv * R) + (size_t)kv * R + jj, sum);
      else agent_store(&part[(size_t)(b0 + bb) * R + jj], sum);
    }
  }
  if constexpr (DEFER == kPushShares) return;
  if constexpr (DEFER) {
    if (wg == 0) {
      for (int b = tid; b < p.B; b += 256) append_defer_bump(p, b, p.seq_lens[b]);
    }
  } else append_finish<R>(p, pl, kv, crow, &flag_sh, n_sh);
}

// ---------------------------------------------------------------- MFMA path: one finishing workgroup per unit
// A unit = (plane, kv head, group of up to SB sequences).  Its contraction over d_model is cut into one LARGE share,
// taken by the unit's finishing workgroup, and NP small ones, taken by helper workgroups (NP = 2: half of d_model, and
// a quarter each; NP = 0: everything in one workgroup).  A helper sums its share and PUSHES the partial tile to the
// finisher as 8-byte words {value, tag} written through to memory; the finisher, busy with twice as much of the factor
// stream, asks for those words before it needs them and finds them valid when its own sum is done, adds them in
// helper order (so the result does not depend on timing), quantises, stores the rows and clears the words again.
// Compared with equal slices merged by "last arriver sums": no ticket, no wait for store acknowledgements, no read-back
// after the last arrival: three dependent memory round trips less on the launch's critical path, while 3 * 2 * Hkv
// workgroups still pull the factor stream instead of 2 * Hkv (a CU sustains only about 70 GB/s of such loads, so one
// workgroup per unit spends 5 us fetching its 384 KB).
// Helpers have the lower workgroup ids of their unit and never wait, so they are dispatched first and always finish;
// the finisher's wait is bounded all the same (WSVD_E_HIP in the status word if a word never arrives).
// Waves split the workgroup's share of d_model; a wave keeps the factor operands of its k-steps in registers
// (requested in two batches around the staging of the hidden states, which all waves copy into LDS with coalesced
// loads); partial tiles meet in LDS (in the hidden states' place) and are summed in wave order.
// DEFER (the decode step's projection launch): NP equal slices of d_model per (plane, kv head), no finisher and no
// hand-off inside the launch: every workgroup leaves its partial sums in p.defer_out, workgroup 0 of each group of
// sequences advances the lengths and marks the rows as pending; the attention launch that follows sums the slices in
// slice order, quantises and stores the rows (the kernel boundary is the hand-off).
// kDeferShares: the same with the shares of the append itself (half, quarter, quarter; partial sum 0 is the half), so that
// the rows are bit for bit the append's: fp32 / bf16 latents.  One sequence of 32 heads, rank 32, d_model 4096: 8.0 us
// against 9.3 us for the launch that finishes the rows itself (four equal slices: 6.9 us, but other bits).
// kPushShares: kDeferShares inside a launch that attends too (wsvd_step.hip): words for the attention's workgroups.
// wg: the workgroup's place among the n_wg of its group of sequences.  Params: by value in a kernel of
// its own (by reference 8 more registers, 0.4 us for 64 sequences), by reference where they are part of a larger kernel argument
// (a copy of that part goes through scratch memory, 16 us a step instead of 11 for one bf16 sequence).
// VW: shares of the contraction per wave, each with accumulators of its own, where the launch has fewer waves than the append
// (the sums are the same: share by share).  A wave asks for the first KB k-steps of all its shares at once.
template <int R, int NT, int DEFER, int VW = 1, class Params = AppendParams>
WSVD_DEV void append_split_body(Params p, int SB, int xs_stride /* elements */, int NP,
                                unsigned long long* ll /* [units][groups][NP][SB * R] */, int wg, int n_wg, int group, int n_groups,
                                uint8_t* app_lds) {
  __shared__ int n_loc[32];
  __shared__ int flag_sh;
  constexpr int RTC = (R + 31) / 32;          // 32-channel row tiles (R = 16 uses half a tile)
  constexpr int KB = 8;                       // k-steps (of 16 model dims) per batch of factor loads
  uint16_t* xs = (uint16_t*)app_lds;                            // [SB][xs_stride] hidden states (bf16)
  float (*red)[R + 1] = (float (*)[R + 1])app_lds;              // [NW * SB][R + 1] partial tiles, later [SB][R + 1] rows
  const int tid = threadIdx.x, lane = tid & 63, wave = tid >> 6, NW = (int)(blockDim.x >> 6) * VW;
  const int n_roles = defer_slices(DEFER) ? NP : NP + 1;
  const int unit = wg / n_roles, role = wg % n_roles;     // role < NP: helper, NP: finisher
  const bool finisher = !DEFER && role == NP, first_share = !defer_slices(DEFER) && role == NP;
  const int pl = unit / p.Hkv, kv = unit % p.Hkv;
  const int b0 = group * SB, nb = min(SB, p.B - b0);
  const int col = lane & 31, g = lane >> 5;
  [[maybe_unused]] const int tl_wg = group * n_wg + wg;
  WSVD_STAMP(p.timeline, tl_wg, wave, 0);
  // the lengths first: nothing depends on them until the rows are stored
  const int nreg = finisher ? append_target_row(p, b0 + min(tid, nb - 1)) : 0;
  // ... and, for the finisher that will turn out to be the last one, the lengths it advances on its way out: asked for
  // now, they cost nothing then (nobody writes them before that)
  int n_bump = (finisher && !p.fused) ? p.seq_lens[p.one_seq >= 0 ? p.one_seq : min(tid, p.B - 1)] : 0;
  if (DEFER && !defer_pushes(DEFER) && wg == 0) n_bump = p.seq_lens[b0 + min(tid, nb - 1)];
  const uint16_t* Ap = (const uint16_t*)p.A[pl];
  const uint16_t* xp = (const uint16_t*)p.x;
  // ---- this workgroup's share of the k-steps (16 model dims each), then this wave's share of that
  const int nks = p.E >> 4;
  const int nks_fin = defer_slices(DEFER) ? 0 : NP ? (nks + 1) / 2 : nks;     // the finisher's share comes first
  const int per_helper = NP ? (nks - nks_fin + NP - 1) / NP : 0;
  const int wg_k0 = first_share ? 0 : min(nks, nks_fin + role * per_helper);
  const int wg_k1 = first_share ? nks_fin : min(nks, wg_k0 + per_helper);
  const int per_wave = (wg_k1 - wg_k0 + NW - 1) / NW;
  int ks0[VW], ks1[VW];
#pragma unroll
  for (int v = 0; v < VW; v++) { ks0[v] = min(wg_k1, wg_k0 + (wave * VW + v) * per_wave); ks1[v] = min(wg_k1, ks0[v] + per_wave); }
  unsigned long long* ll_unit = ll + ((size_t)(unit * n_groups + group) * (NP ? NP : 1)) * (size_t)(SB * R);
  constexpr int NB = VW == 1 ? 2 : VW;        // batches in flight: two of the one share, or one of each
  v8bf aop[NB][RTC][KB];
  // Only the k-steps of the wave's own part are requested (wave-uniform predicate): the CU's address pipeline moves
  // 64 bytes per clock, and with 16 waves asking for everything at once every surplus request delays the useful ones.
  auto load_a = [&](int buf, int k0) {
    const int end = ks1[VW == 1 ? 0 : buf];
#pragma unroll
    for (int k = 0; k < KB; k++) {
      if (k0 + k < end) {
#pragma unroll
        for (int rt = 0; rt < RTC; rt++)
          aop[buf][rt][k] = *(const v8bf*)(Ap + (((size_t)(kv * RTC + rt) * (size_t)nks + (size_t)(k0 + k)) * 64 + lane) * 8);
      }
    }
  };
  // ---- in the int8 step of one launch: the factors of the first k-steps, and behind them the share of the hidden states
  // straight to LDS, 1 KiB of a row per instruction, dealt to the waves: all of it in flight at once, without a register.
  // The few workgroups of that launch are bound by this round trip, which the attention's waves wait for: four layers of 16
  // heads, one sequence of 500 rows 44.7 -> 41.7 us, three of 2048 50.4 -> 48.1.  Everywhere else it is no gain or a loss
  // (the bf16 step 90.0 -> 90.5 us, 64 sequences of 300 rows in two launches 30.8 -> 31.9, 28 heads on 4 93.7 -> 95.7: the
  // workgroups that share a CU hide the trip, and the registers' copies start the products earlier), so that the pieces
  // go through registers there.
  if constexpr (DEFER == kPushSlices) {
    static_assert(VW == 1);
    load_a(0, ks0[0]); load_a(1, ks0[0] + KB);
    const int ppr = (wg_k1 - wg_k0) * 2, segs = (ppr + 63) >> 6, n_segs = nb * segs;   // pieces of 16 bytes, instructions per row
    const uint32_t lds0 = __builtin_amdgcn_readfirstlane(lds_address(app_lds));
    for (int i = __builtin_amdgcn_readfirstlane(wave); i < n_segs; i += (int)(blockDim.x >> 6)) {
      const int row = i / segs, seg = i - row * segs;
      const uint8_t* src = (const uint8_t*)(xp + (size_t)(b0 + row) * p.E + (size_t)wg_k0 * 16) + seg * 1024;
      if (seg * 64 + lane < ppr) lds_copy16(lds0 + row * xs_stride * 2 + seg * 1024, src, lane * 16);
    }
    WSVD_STAMP(p.timeline, tl_wg, wave, 1);
    asm volatile("s_waitcnt vmcnt(0)" ::: "memory");
  } else {
    // Otherwise: hidden states of the share -> LDS, whole 16-byte pieces, kPieces per thread and trip in flight (wave-uniform
    // predicate per piece); the factor batches go out between the first trip's requests and its LDS writes, so that a
    // wave's first k-steps cost one round trip.  The row of piece i is i / ppr by a reciprocal: (i + 1/2) / ppr is at least
    // 1 / (2 ppr) away from every integer, more than the product is off (a row number below 32 times 2^-22; ppr < 2^13, or the
    // row is 0), so its integer part is exact.  Two integer divisions per piece / one
    // per thread and a walk from piece to piece / this, append + attention over 130 cached rows: 64 sequences of 32 heads,
    // int8, 31.5 / 30.2 / 29.4 us, 23 paged ones 20.7 / 20.0 / 19.6, one sequence of 8 heads, d_model 512, 10.9 / 11.1 / 10.9.
    // Eight pieces in flight: 0.5 us less for 64 sequences, but 0.5 to 4 us more for up to 32 and for the slices of the int8
    // step (registers).
    constexpr int kPieces = 4;
    const int ppr = (wg_k1 - wg_k0) * 2, n_pieces = nb * ppr;     // 16-byte pieces per row (none: an empty share)
    const float per_row = __builtin_amdgcn_rcpf((float)ppr);
    bool first = true;
    for (int i0 = 0; i0 < n_pieces || first; i0 += kPieces * (int)blockDim.x) {
      v4i piece[kPieces];
      int to[kPieces];                                            // LDS element of the piece
#pragma unroll
      for (int it = 0; it < kPieces; it++) {
        if (i0 + it * (int)blockDim.x + (wave << 6) < n_pieces) { // some lane of this wave has a piece
          const int i = min(i0 + it * (int)blockDim.x + tid, n_pieces - 1);
          const int row = (int)(((float)i + 0.5f) * per_row), at = (i - row * ppr) * 8;
          piece[it] = *(const v4i*)(xp + (size_t)(b0 + row) * p.E + (size_t)wg_k0 * 16 + at);
          to[it] = row * xs_stride + at;
        }
      }
      if (first) {
        if constexpr (VW == 1) { load_a(0, ks0[0]); load_a(1, ks0[0] + KB); }
        else {
#pragma unroll
          for (int v = 0; v < VW; v++) load_a(v, ks0[v]);
        }
        first = false; WSVD_STAMP(p.timeline, tl_wg, wave, 1);
      }
#pragma unroll
      for (int it = 0; it < kPieces; it++)
        if (i0 + it * (int)blockDim.x + tid < n_pieces) *(v4i*)&xs[to[it]] = piece[it];
    }
  }
  if (tid < 32) n_loc[tid] = nreg;
  __syncthreads();
  WSVD_STAMP(p.timeline, tl_wg, wave, 2);
  // every user of the old lengths draws a ticket once it holds them; whoever draws the last one advances them
  const int ticket = (tid == 0 && finisher && !p.fused) ? append_reader_ticket(p) : 0;
  v16f acc[VW][RTC];
#pragma unroll
  for (int w = 0; w < VW; w++)
#pragma unroll
    for (int rt = 0; rt < RTC; rt++)
#pragma unroll
      for (int v = 0; v < 16; v++) acc[w][rt][v] = 0.f;
  const uint16_t* xrow = xs + (size_t)min(col, nb - 1) * xs_stride + g * 8;   // columns past the group repeat its last row
  auto mul = [&](int buf, int k0) {
    const int w = VW == 1 ? 0 : buf;
#pragma unroll
    for (int k = 0; k < KB; k++)
      if (k0 + k < ks1[w]) {                                       // wave-uniform
        const v8bf xo = *(const v8bf*)(xrow + (k0 + k - wg_k0) * 16);
#pragma unroll
        for (int rt = 0; rt < RTC; rt++) acc[w][rt] = __builtin_amdgcn_mfma_f32_32x32x16_bf16(aop[buf][rt][k], xo, acc[w][rt], 0, 0, 0);
      }
  };
  if constexpr (VW == 1) {
    for (int k0 = ks0[0]; k0 < ks1[0]; k0 += 2 * KB) {
      mul(0, k0);
      if (k0 + 2 * KB < ks1[0]) load_a(0, k0 + 2 * KB);         // (wave-uniform; nothing is requested past the wave's part)
      mul(1, k0 + KB);
      if (k0 + 3 * KB < ks1[0]) load_a(1, k0 + 3 * KB);
    }
  } else {
    for (int o = 0; o < per_wave; o += KB)
#pragma unroll
      for (int v = 0; v < VW; v++) {
        mul(v, ks0[v] + o);
        if (o + KB < per_wave) load_a(v, ks0[v] + o + KB);
      }
  }
  WSVD_STAMP(p.timeline, tl_wg, wave, 3);
  // the finisher asks for the helpers' words now, one (sequence, channel) element per thread and helper: whatever
  // has arrived by the time its own sum is done needs no second look
  constexpr int NPMAX = 2, EPT = (32 * R + NT - 1) / NT;         // helpers; elements per thread (SB <= 32)
  unsigned long long w[EPT][NPMAX];
  if (finisher && NP) {
#pragma unroll
    for (int e = 0; e < EPT; e++) {
      const int i = min(tid + e * (int)blockDim.x, SB * R - 1);
#pragma unroll
      for (int h = 0; h < NPMAX; h++)
        w[e][h] = __hip_atomic_load(ll_unit + (size_t)min(h, NP - 1) * (SB * R) + i, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT);
    }
  }
  __syncthreads();                                              // the hidden states are no longer read: their LDS is reused
#pragma unroll
  for (int w = 0; w < VW; w++)
#pragma unroll
    for (int rt = 0; rt < RTC; rt++)
#pragma unroll
      for (int v = 0; v < 16; v++) {
        // lane holds sequence column `col`, channel rows 8*(v/4) + 4*g + v%4
        const int ch = rt * 32 + 8 * (v / 4) + 4 * g + (v % 4);
        if (ch < R && col < nb) red[(wave * VW + w) * SB + col][ch] = acc[w][rt][v];
      }
  __syncthreads();
  WSVD_STAMP(p.timeline, tl_wg, wave, 4);
  // sum over the waves in wave order, one thread per (sequence, channel); the result replaces wave 0's partial, which
  // only this thread reads
#pragma unroll
  for (int e = 0; e < EPT; e++) {
    const int i = tid + e * (int)blockDim.x;
    if (i < nb * R) {
      const int row = i / R, j = i % R;
      float c = 0.f;
      for (int k = 0; k < NW; k++) c += red[k * SB + row][j];
      if constexpr (DEFER) {
        const int part = defer_slices(DEFER) ? role : first_share ? 0 : role + 1;
        append_defer_out<DEFER>(p, (((size_t)part * 2 + pl) * p.B + b0 + row) * ((size_t)p.Hkv * R) + (size_t)kv * R + j, c);
      } else if (!finisher) {
        // push: value and tag in one 8-byte store, written through; nobody waits for it
        __hip_atomic_store(ll_unit + (size_t)role * (SB * R) + (size_t)row * R + j, ll_word(c), __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT);
      } else {
        if (NP) {
          unsigned long long* src = ll_unit + (size_t)row * R + j;
#pragma unroll
          for (int h = 0; h < NPMAX; h++) {
            if (h < NP) {
              unsigned long long v = w[e][h];
              int budget = 1 << 16;
              while ((uint32_t)(v >> 32) != kLLTag && budget > 0) {
                __builtin_amdgcn_s_sleep(1);
                v = __hip_atomic_load(src + (size_t)h * (SB * R), __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT);
                budget--;
              }
              if ((uint32_t)(v >> 32) != kLLTag) atomicExch(p.err_word, (int)WSVD_E_HIP);   // never seen; keeps the kernel finite
              c += __uint_as_float((uint32_t)v);
              // cleared for the next launch (a kernel boundary lies between); written through like the push itself
              __hip_atomic_store(src + (size_t)h * (SB * R), 0ull, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT);
            }
          }
        }
        red[row][j] = c;
      }
    }
  }
  if constexpr (DEFER) {
    if (!defer_pushes(DEFER) && wg == 0 && tid < nb) append_defer_bump(p, b0 + tid, n_bump);
    WSVD_STAMP(p.timeline, tl_wg, wave, 5);
    return;
  }
  if (!finisher) return;
  __syncthreads();
  WSVD_STAMP(p.timeline, tl_wg, wave, 5);
  append_store_rows<R>(p, pl, kv, b0, nb, red, n_loc - b0);
  WSVD_STAMP(p.timeline, tl_wg, wave, 6);
  if (p.fused) return;
  // ---- the lengths: advanced by the last finisher to have drawn a ticket (all others hold their copies by then)
  __syncthreads();
  if (tid == 0) {
    const int last = (ticket == n_wg / (NP + 1) * n_groups - 1);
    if (last) __hip_atomic_store(p.tickets + 2 * p.Hkv, 0, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT);
    flag_sh = last;
  }
  __syncthreads();
  if (!flag_sh) return;
  if (p.one_seq >= 0) {
    if (tid == 0) {
      const int n0 = n_bump;
      if (n0 >= 0) p.seq_lens[p.one_seq] = min(n0 + p.B, p.t_cap);
      if (n0 < 0 || n0 + p.B > p.t_cap) atomicExch(p.err_word, (int)WSVD_E_CAPACITY);
    }
    return;
  }
  for (int b = tid; b < p.B; b += blockDim.x) {
    const int n = b == tid ? n_bump : p.seq_lens[b];            // (more sequences than threads: the rest is read now)
    if (n >= 0 && n < p.t_cap) p.seq_lens[b] = n + 1;
    else atomicExch(p.err_word, (int)WSVD_E_CAPACITY);
  }
}
