// Decode attention over F32 / BF16 latent caches (row-major planes), plain vector ALU.
//
// A latent row is rank*esize bytes; LPR = row_bytes/16 adjacent lanes share a row, each holding a
// 16-byte slice, so a wavefront load covers 64/LPR consecutive rows = 1 KiB of contiguous cache.
// Each lane group runs its own online softmax (running max, sum, latent-space accumulator) over the
// rows it streams; the groups are merged once at the end, like sequence splits.
#pragma once
#include "wsvd_attn_common.h"
#include "wsvd_append_split.h"

template <int ESZ>
WSVD_DEV void unpack16(const v4i& raw, float* f) {
  if (ESZ == 4) {
#pragma unroll
    for (int i = 0; i < 4; i++) f[i] = __int_as_float(raw[i]);
  } else {
#pragma unroll
    for (int i = 0; i < 4; i++) {
      f[2 * i] = __uint_as_float((uint32_t)raw[i] << 16);
      f[2 * i + 1] = __uint_as_float((uint32_t)raw[i] & 0xFFFF0000u);
    }
  }
}

// The new row of (sequence b, kv head) from the words of the launch's projection workgroups: element tid % R of the K latent
// (tid < R) or of the V latent (tid < 2 R), the parts added in slice order.  All that exist are asked for at once, eight at a
// time, and again until they carry the tag; then they are cleared for the next launch.  The workgroups waited for have lower
// ids and wait for nothing; the wait is bounded all the same.
template <int R>
WSVD_DEV float step_row_sum(const AttnParams& p, int kv, int b) {
  const int tid = threadIdx.x;
  if (tid >= 2 * R) return 0.f;
  constexpr int AT_ONCE = 8;
  unsigned long long* const src = p.new_words + (size_t)(tid / R) * (p.part_stride / 2) + (size_t)b * p.new_ld + (size_t)kv * R + tid % R;
  float c = 0.f;
  for (int i0 = 0; i0 < p.n_parts; i0 += AT_ONCE) {
    unsigned long long w[AT_ONCE];
    int budget = 1 << 16;
    for (;;) {
#pragma unroll
      for (int i = 0; i < AT_ONCE; i++)
        if (i == 0 || i0 + i < p.n_parts)                        // (uniform)
          w[i] = __hip_atomic_load(src + (size_t)(i0 + i) * p.part_stride, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT);
        else w[i] = w[0];
      bool all = true;
#pragma unroll
      for (int i = 0; i < AT_ONCE; i++) all = all && (uint32_t)(w[i] >> 32) == kLLTag;
      if (all) break;
      if (--budget == 0) { atomicExch(p.err_word, (int)WSVD_E_HIP); break; }     // never seen; keeps the wait finite
      __builtin_amdgcn_s_sleep(1);
    }
#pragma unroll
    for (int i = 0; i < AT_ONCE; i++)
      if (i == 0 || i0 + i < p.n_parts) {
        c += __uint_as_float((uint32_t)w[i]);
        __hip_atomic_store(src + (size_t)(i0 + i) * p.part_stride, 0ull, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT);
      }
  }
  return c;
}

// NEWROW = kRowPending: the second launch of the decode step.  The projection launch before it has advanced the lengths and left the new
// token's latents as n_parts partial sums (p.new_k / p.new_v); the workgroup whose chunk holds a sequence's last row sums
// them in slice order, rounds to the storage format, stores the row and attends to it from LDS, in the place it would
// have in the stream.  The partial sums are asked for with the first loads of the kernel and waited for with the factor.
// NEWROW = kRowWords: the decode step as one launch (wsvd_step.hip).  The lengths are still the old ones (n_raw: the new one),
// the partial sums arrive as {value, tag} words while the chunk is streamed; the workgroup whose chunk ends with the
// sequence's last row waits for them when its stream is over and clears them.
// The first 256 threads of a workgroup work here, whatever its size.
enum { kNoRow = 0, kRowPending = 1, kRowWords = 2 };
template <int ESZ, int R, int G, int NEWROW>
WSVD_DEV void attn_generic_body(const AttnParams& p, int n_raw, int wi_kv, int wi_chunk, int wi_b, bool store_row) {
  constexpr int ROWB = R * ESZ;          // bytes per latent row
  constexpr int LPR = ROWB / 16;         // lanes per row
  constexpr int VPL = 16 / ESZ;          // values per lane
  constexpr int RPW = 64 / LPR;          // rows per wavefront load
  constexpr int NGRP = 4 * RPW;          // lane groups per workgroup
  constexpr int UNROLL = 4;

  constexpr int FIT = R * ESZ / 32;     // 16-byte staging passes for an R x 128 factor
  __shared__ v4i fac_lds[R * 128 * ESZ / 16];
  __shared__ __attribute__((aligned(16))) float q_lds[G * 128];
  __shared__ float qts[G * R];
  __shared__ float Msh[G], Lsh[G], Ush[G * R];
  __shared__ float gm[NGRP * G], gl[NGRP * G];
  __shared__ float gu[NGRP * G * R];
  // parts the merge of the NGRP lane groups is divided into (a power of two that divides NGRP; 1 = a single pass)
  constexpr int NPART = G * R >= 256 ? 1 : (256 / (G * R) >= 8 ? 8 : 256 / (G * R) >= 4 ? 4 : 2);
  static_assert(NGRP % NPART == 0, "the lane groups divide evenly over the parts");
  __shared__ float pm[NPART * G], pl[NPART * G], pu[NPART * G * R];
  __shared__ int flag_sh;

  const int tid = threadIdx.x, lane = tid & 63, wave = tid >> 6;
  // partial sums in flight from the start (fp32 has d_model / 256 of them, where 256 divides it, otherwise up to
  // d_model / 64), and in each batch of further ones.  One after the other: two fp32 sequences of 8 heads, rank 64,
  // d_model 4160, 61.4 us a step, eight at a time 51.9 (the append and the attention call 57.6); 32 heads, rank 32,
  // d_model 4096: 31.0 -> 28.8
  constexpr int MAXP = NEWROW == kRowPending ? 4 : 1, MORE = 8;
  __shared__ float new_row[2][NEWROW ? R : 1];
  [[maybe_unused]] const int pend = NEWROW == kRowPending ? p.pending[wi_b] : 0;
  [[maybe_unused]] float np[MAXP];
  [[maybe_unused]] const float* const np_src = (tid / R ? p.new_v : p.new_k) + (size_t)wi_b * p.new_ld + (size_t)wi_kv * R + tid % R;
  if constexpr (NEWROW == kRowPending) {
    if (tid < 2 * R) {
#pragma unroll
      for (int i = 0; i < MAXP; i++) np[i] = np_src[(size_t)min(i, p.n_parts - 1) * p.part_stride];
    }
  }
  const WorkItem w = decode_work(p, n_raw, wi_kv, wi_chunk, wi_b);
  if constexpr (NEWROW == kRowWords) {
    if (w.n == 0 && w.chunk == 0) step_row_sum<R>(p, wi_kv, wi_b);     // (a negative length: nothing is stored, the words go)
  }
  if (w.n == 0) { write_zero_outputs<256>(p, w); return; }
  if (!w.active) return;
  const int sl = lane % LPR;                       // which 16-byte slice of the row
  const int grp = wave * RPW + lane / LPR;         // lane group id within the workgroup

  const int fac16 = R * p.d * ESZ / 16;
  {
    StageRegs<FIT> st;
    QRegsT<(G * 128 + 255) / 256> qr;               // 256 query elements per pass
    stage_issue<FIT, 256>(st, (const char*)p.BK + (size_t)w.kv * R * p.d * ESZ, fac16);
    q_issue(p, w.b, w.kv, qr);
    stage_commit<FIT, 256>(st, fac_lds, fac16);
    q_commit(p, qr, q_scale_value(p, w.b, q_scale_raw(p, w.b)), q_lds);
  }
  const size_t plane = ((size_t)w.b * p.Hkv + w.kv) * (size_t)p.t_cap * ROWB;
  int row_end = w.row_end;                         // of the rows that are read from the cache
  [[maybe_unused]] bool own_new = false;           // the new row is one of this chunk's
  // the row in the cache's format, in its plane and in LDS
  [[maybe_unused]] auto put_row = [&](float c, int row) {
    uint8_t* dst = const_cast<uint8_t*>(tid / R ? p.v_codes : p.k_codes) + plane + (size_t)row * ROWB;
    if constexpr (ESZ == 4) ((float*)dst)[tid % R] = c;
    else {
      const uint16_t h = f32_to_bf16_rne(c);
      ((uint16_t*)dst)[tid % R] = h;
      c = bf16_to_f32(h);
    }
    new_row[tid / R][tid % R] = c;
  };
  // (a sequence longer than the caller's bound is reported by decode_work; its row is still stored, by the last chunk)
  [[maybe_unused]] const bool last_chunk = w.chunk == min((w.n - 1) / p.chunk_rows, p.n_chunks - 1);
  if constexpr (NEWROW == kRowWords) {
    own_new = store_row && last_chunk && w.n - 1 < w.row_end;
    row_end = own_new ? w.n - 1 : w.row_end;
  }
  if constexpr (NEWROW == kRowPending) {
    const int row = w.n - 1;
    if (pend != 0 && last_chunk) {
      own_new = row < w.row_end;
      row_end = own_new ? row : w.row_end;
      if (tid < 2 * R) {
        float c = np[0];
#pragma unroll
        for (int i = 1; i < MAXP; i++) c += i < p.n_parts ? np[i] : 0.f;
        for (int i0 = MAXP; i0 < p.n_parts; i0 += MORE) {
          float more[MORE];
#pragma unroll
          for (int i = 0; i < MORE; i++) more[i] = np_src[(size_t)min(i0 + i, p.n_parts - 1) * p.part_stride];
#pragma unroll
          for (int i = 0; i < MORE; i++) c += i0 + i < p.n_parts ? more[i] : 0.f;
        }
        put_row(c, row);
      }
    }
  }
  __syncthreads();
  compute_qtilde<R, ESZ, 256>(p, fac_lds, q_lds, qts);
  float qt[G][VPL];
#pragma unroll
  for (int g = 0; g < G; g++)
#pragma unroll
    for (int v = 0; v < VPL; v++) qt[g][v] = qts[g * R + sl * VPL + v];

  const uint8_t* kb = p.k_codes + plane + sl * 16;
  const uint8_t* vb = p.v_codes + plane + sl * 16;

  float m[G], l[G], u[G][VPL];
#pragma unroll
  for (int g = 0; g < G; g++) {
    m[g] = -INFINITY; l[g] = 0.f;
#pragma unroll
    for (int v = 0; v < VPL; v++) u[g][v] = 0.f;
  }

  // Two batches of UNROLL rows per lane group in flight: the next batch is requested before the current one is
  // consumed, so a short chunk (640 rows = 3 batches) waits for memory twice, not three times: 8.3 -> 7.9 us for the
  // single 640-row bf16 sequence.  Rows are consumed in the same order as without the prefetch.  (Measured slower:
  // the first batches and B_V requested in front of the query absorption, 8.5-8.9 us.)
  constexpr int STEP = NGRP * UNROLL;
  auto load_rows = [&](v4i (&kr)[UNROLL], v4i (&vr)[UNROLL], int t0) {
#pragma unroll
    for (int k = 0; k < UNROLL; k++) {
      const int t = t0 + k * NGRP;
      if (t < row_end) {
        kr[k] = *(const v4i*)(kb + (size_t)t * ROWB);
        vr[k] = *(const v4i*)(vb + (size_t)t * ROWB);
      }
    }
  };
  auto use_row = [&](const float (&kf)[VPL], const float (&vf)[VPL]) {
#pragma unroll
    for (int g = 0; g < G; g++) {
      float s = 0.f;
#pragma unroll
      for (int v = 0; v < VPL; v++) s = fmaf(qt[g][v], kf[v], s);
      s = group_sum<LPR>(s);
      const float mn = fmaxf(m[g], s);
      const float alpha = __builtin_amdgcn_exp2f(m[g] - mn);
      const float pw = __builtin_amdgcn_exp2f(s - mn);
      l[g] = fmaf(l[g], alpha, pw);
#pragma unroll
      for (int v = 0; v < VPL; v++) u[g][v] = fmaf(u[g][v], alpha, pw * vf[v]);
      m[g] = mn;
    }
  };
  auto use_rows = [&](const v4i (&kr)[UNROLL], const v4i (&vr)[UNROLL], int t0) {
#pragma unroll
    for (int k = 0; k < UNROLL; k++) {
      const int t = t0 + k * NGRP;
      if (t < row_end) {            // uniform within a lane group
        float kf[VPL], vf[VPL];
        unpack16<ESZ>(kr[k], kf);
        unpack16<ESZ>(vr[k], vf);
        use_row(kf, vf);
      }
    }
  };
  {
    v4i ka[UNROLL], va[UNROLL], kb2[UNROLL], vb2[UNROLL];
    int t0 = w.row_begin + grp;
    load_rows(ka, va, t0);
    while (t0 < row_end) {
      load_rows(kb2, vb2, t0 + STEP);       // (nothing is requested past the chunk's end)
      use_rows(ka, va, t0);
      t0 += STEP;
      if (t0 >= row_end) break;
      load_rows(ka, va, t0 + STEP);
      use_rows(kb2, vb2, t0);
      t0 += STEP;
    }
  }
  // B_V is asked for here: its trip to memory runs beside the merge, and beside the wait for the new row
  StageRegs<FIT> stv;
  stage_issue<FIT, 256>(stv, (const char*)p.BV + (size_t)w.kv * R * p.d * ESZ, fac16);
  if constexpr (NEWROW == kRowWords) {
    if (last_chunk) {
      const float c = step_row_sum<R>(p, wi_kv, wi_b);
      if (store_row && tid < 2 * R) put_row(c, w.n - 1);
      __syncthreads();
    }
  }
  if constexpr (NEWROW) {
    if (own_new && (w.n - 1 - w.row_begin) % NGRP == grp) {             // the lane group whose turn the row is
      float kf[VPL], vf[VPL];
#pragma unroll
      for (int v = 0; v < VPL; v++) { kf[v] = new_row[0][sl * VPL + v]; vf[v] = new_row[1][sl * VPL + v]; }
      use_row(kf, vf);
    }
  }
  // NOTE: group_sum uses DPP across the LPR lanes of a row; lanes of a group take the same branch
  // (t depends only on the group), so the exchanged values are always defined.

#pragma unroll
  for (int g = 0; g < G; g++) {
    if (sl == 0) { gm[grp * G + g] = m[g]; gl[grp * G + g] = l[g]; }
#pragma unroll
    for (int v = 0; v < VPL; v++) gu[(grp * G + g) * R + sl * VPL + v] = u[g][v];
  }
  __syncthreads();
  // Merge of the lane groups' partial results, one thread per (part of the groups, head, latent dim), then one per
  // (head, latent dim) over the parts: with a single head of rank 32 a lone pass would leave 224 of the 256 threads idle
  // while 32 walk 64 groups each.
  if constexpr (NPART > 1) {
    for (int i = tid; i < NPART * G * R; i += 256) {
      const int part = i / (G * R), g = (i / R) % G, j = i % R;
      const int k0 = part * (NGRP / NPART), k1 = k0 + NGRP / NPART;
      float M = -INFINITY;
      for (int k = k0; k < k1; k++) M = fmaxf(M, gm[k * G + g]);
      float L = 0.f, U = 0.f;
      for (int k = k0; k < k1; k++) {
        const float e = M == -INFINITY ? 0.f : __builtin_amdgcn_exp2f(gm[k * G + g] - M);   // a part without any row
        L = fmaf(gl[k * G + g], e, L);
        U = fmaf(gu[(k * G + g) * R + j], e, U);
      }
      pu[i] = U;
      if (j == 0) { pm[part * G + g] = M; pl[part * G + g] = L; }
    }
    __syncthreads();
  }
  for (int i = tid; i < G * R; i += 256) {
    const int g = i / R, j = i % R;
    const float* sm = NPART > 1 ? pm : gm;
    const float* sl_ = NPART > 1 ? pl : gl;
    const float* su = NPART > 1 ? pu : gu;
    constexpr int NS = NPART > 1 ? NPART : NGRP;
    float M = -INFINITY;
    for (int k = 0; k < NS; k++) M = fmaxf(M, sm[k * G + g]);
    float L = 0.f, U = 0.f;
    for (int k = 0; k < NS; k++) {
      const float e = __builtin_amdgcn_exp2f(sm[k * G + g] - M);      // the workgroup holds at least one row: M is finite
      L = fmaf(sl_[k * G + g], e, L);
      U = fmaf(su[(k * G + g) * R + j], e, U);
    }
    Ush[i] = U;
    if (j == 0) { Msh[g] = M; Lsh[g] = L; }
  }
  stage_commit<FIT, 256>(stv, fac_lds, fac16);     // B_K is no longer needed: its LDS holds B_V from here on
  __syncthreads();
  attn_tail<R, ESZ, 256>(p, w, Msh, Lsh, Ush, &flag_sh, fac_lds);
}
