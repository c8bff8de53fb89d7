// The decode step over fp32 / bf16 latents as ONE launch: projection workgroups and attention workgroups side by side.
//
// For a few short sequences both halves of the step are chains of memory round trips with the chip nearly empty, and
// neither needs the other until the new row is attended to.  So workgroups [0, n_proj) run the append's projection and push
// their partial sums as {value, tag} words (kPushShares); the others stream the cached rows as wsvd_decode_attn does,
// and the one whose chunk holds a sequence's last row takes the words when its stream is over, sums them in the append's order,
// rounds and stores the row and attends to it (kRowWords).  Rows and outputs are those of the two launches bit for bit.
// Bound: the projection's chain (one trip for its factors, the sum over the waves), one hand-off, the attention's merge and B_V.
//
// Who waits for whom: attention for projection workgroups, which have the lower ids and wait for nothing; of each sequence the
// workgroup with the highest id for the others' word that they have read the old length, which it then advances.  All waits
// are bounded.
#include "wsvd_attn_generic_body.h"
#include "wsvd_internal.h"

struct FloatStepParams {
  AttnParams a;
  AppendParams ap;
  int n_proj;                  // projection workgroups
  int* read;                   // [B] workgroups that have read the sequence's length; zero between launches
  // bf16 latents: the shape of append_split_body
  int xs_stride, helpers;
};

template <int ESZ, int R, int G>
WSVD_DEV void step_attend(const FloatStepParams& p) {
  const AttnParams& a = p.a;
  if (threadIdx.x >= 256) return;
  const int id = (int)blockIdx.x - p.n_proj;
  const int kv = id % a.Hkv, chunk = id / a.Hkv % a.n_chunks, b = id / (a.Hkv * a.n_chunks);
  int n = a.seq_lens[b];
  asm volatile("" : "+s"(n)::"memory");                          // this wave holds the length ...
  __syncthreads();                                               // ... and so do the other three: their workgroup may be counted
  const bool fits = n >= 0 && n < a.t_cap;
  if (threadIdx.x == 0) __hip_atomic_fetch_add(p.read + b, 1, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT);
  attn_generic_body<ESZ, R, G, kRowWords>(a, fits ? n + 1 : n, kv, chunk, b, fits);
  if (kv != a.Hkv - 1 || chunk != a.n_chunks - 1 || threadIdx.x != 0) return;
  const int want = a.Hkv * a.n_chunks;
  int budget = 1 << 16;
  while (__hip_atomic_load(p.read + b, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT) != want && --budget > 0) __builtin_amdgcn_s_sleep(8);
  if (budget == 0) atomicExch(a.err_word, (int)WSVD_E_HIP);      // never seen; keeps the wait finite
  __hip_atomic_store(p.read + b, 0, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT);
  if (fits) p.ap.seq_lens[b] = n + 1;
  else atomicExch(a.err_word, (int)WSVD_E_CAPACITY);
}

template <int R, int G, int NT, int VW>
__global__ __launch_bounds__(NT) void k_step_bf16(FloatStepParams p) {
  extern __shared__ __align__(16) uint8_t app_lds[];
  if ((int)blockIdx.x < p.n_proj) append_split_body<R, NT, kPushShares, VW, const AppendParams&>(p.ap, p.ap.B, p.xs_stride, p.helpers, nullptr, (int)blockIdx.x, p.n_proj, 0, 1, app_lds);
  else step_attend<2, R, G>(p);
}
template <int R, int G, int BB>
__global__ __launch_bounds__(256) void k_step_f32(FloatStepParams p) {
  if ((int)blockIdx.x < p.n_proj) append_valu_body<R, 4, kPushShares, BB, const AppendParams&>(p.ap, (int)blockIdx.x);
  else step_attend<4, R, G>(p);
}

// Shares of the projection per wave.  Two: 8 waves where the append has 16 (rank 64: 4 for 8), so that the attention has 256
// registers a lane; with one, a group of 4 query heads spilled 122 of them (8 kv heads, rank 32, 900 rows: 30.5 us, now 17.44).
constexpr int kStepShares = 2;
constexpr int kStepLds = 40 * 1024;      // limit of the projection's hidden states and partial sums

// One launch or two.  One gains while both halves find room beside each other; beyond that the attention has fewer waves per CU
// than in a launch of its own, and its stream is the time.  us a step, one launch / two, replayed from a graph over cold layers:
//   bf16  1 sequence x 900 rows, 32 heads, rank 32, E = d_model 4096   12.9 / 18.2
//   bf16  4 x 900, the same                                            15.4 / 18.9
//   bf16  8 x 900, 8 kv heads of 4, rank 32                            18.3 / 23.8
//   bf16  4 x 234, 8 kv heads of 7, rank 16, E 7168                    19.1 / 20.7
//   bf16  8 x 8000, 8 kv heads of 4, rank 32 (beyond)                  45.7 / 38.0
//   bf16  16 x 8000, 8 heads, rank 16, E 512 (beyond)                  29.4 / 25.8
//   fp32  1 x 250, 8 heads, rank 16, E 512                             7.4 / 9.5
//   fp32  64 x 900, 8 heads, rank 64, E 512                            92.0 / 123.8
//   fp32  4 x 8000, 32 heads, rank 16, E 4096 (beyond)                 54.3 / 45.8
//   fp32  16 x 8000, 4 kv heads of 7, rank 64, E 3584 (beyond)         139 / 112
// A projection that outlasts the rows' stream is better off alone.  bf16: a wave has two of the append's shares here, and where a
// share is more than the one batch of 8 k-steps that the wave asks for at once, the rows have to make up for it:
//   3 x 23 rows, 8 heads, rank 16, E 7168           13.2 / 12.1     4 x 1164, the same             15.2 / 15.5
//   8 x 3, 4 heads of 64, rank 64, E 4096           14.3 / 13.1     1 x 10, 8 kv heads of 2        11.6 / 13.8
//   1 x 15, 1 head, rank 16, E 16384                22.8 / 14.4     1 x 490, 12 kv heads of 2, rank 32, E 5120   11.3 / 15.0
// fp32: many partial sums are as many words for one workgroup to take, and with more than 4 query heads an attention workgroup has
// no place until the projection's leave:
//   2 x 4299, 1 kv head of 2, rank 16, E 8128 (127 sums)   27.6 / 20.5
//   28 x 8, 8 kv heads of 7, rank 16, E 7168        33.0 / 30.7     4 x 96, the same               19.1 / 20.6
// Of 9242 bf16 sizes on this side of the lines (1 to 32 kv heads, d_model 512 to 12288, 1 to 8192 rows) the median is 1.20 x, one in a
// hundred below 0.984, the worst 0.915; of 1388 fp32 sizes 1.18, 0.961 and 0.91.  Beyond them the median is 0.96 for both.
// Groups of 7 gain although those of ranks 16 and 32 spill 25 registers.  Groups of 8 are not chosen, only built (they would gain
// too: 359 sizes of 2 kv heads, d_model 1024, median 1.11 x).
static bool step_one_launch(const wsvd_ctx* ctx, const wsvd_layer_desc& d, const FloatStepParams& p, int waves, int attend, int max_seq_len) {
  const int G = d.n_q_heads / d.n_kv_heads, rows = max_seq_len < p.a.chunk_rows ? max_seq_len : p.a.chunk_rows;
  if (d.latent_dtype == WSVD_BF16) {
    if (G == 8 || p.n_proj + 2 * attend > 2 * ctx->n_cu) return false;
    const int steps = ((p.helpers ? (d.d_model / 16 + 1) / 2 : d.d_model / 16) + waves - 1) / waves, batches = (steps + 7) / 8;
    if (d.rank < 64) return steps <= 12 || (steps <= 24 && rows * G * d.rank >= 16 * 512 * (steps - 12));
    return batches <= 1 || (batches <= 6 && (G > 1 || rows >= 32 << batches || (batches == 2 && 2 * p.n_proj > ctx->n_cu)));
  }
  if (p.a.n_parts > 40 + G * d.rank / 4 || (G > 4 && p.n_proj > ctx->n_cu && p.n_proj + attend > 2 * ctx->n_cu)) return false;
  return p.n_proj <= 2 * ctx->n_cu && attend <= (d.rank == 64 && G > 4 ? 1 : 4) * ctx->n_cu;   // (72 KB of LDS and more)
}

template <int R, int G>
static hipError_t launch_step(const FloatStepParams& p, int latent_dtype, size_t lds, hipStream_t s) {
  const dim3 grid((unsigned)(p.n_proj + p.a.Hkv * p.a.n_chunks * p.a.B));
  constexpr int VW = kStepShares, NT = (R == 64 ? 512 : 1024) / VW;
  if (latent_dtype == WSVD_BF16) {
    static LdsLimit limit;                                       // (with the attention's arrays of rank 64 above 64 KB)
    hipError_t e = wsvd_raise_lds(limit, (const void*)k_step_bf16<R, G, NT, VW>, kStepLds);
    if (e != hipSuccess) return e;
    hipLaunchKernelGGL((k_step_bf16<R, G, NT, VW>), grid, dim3(NT), lds, s, p);
  } else if (p.a.B == 1) hipLaunchKernelGGL((k_step_f32<R, G, 1>), grid, dim3(256), 0, s, p);
  else hipLaunchKernelGGL((k_step_f32<R, G, kAppendBB>), grid, dim3(256), 0, s, p);
  return hipGetLastError();
}
template <int R>
static hipError_t launch_step_g(const FloatStepParams& p, int latent_dtype, size_t lds, hipStream_t s) {
  switch (p.a.G) {
    case 1: return launch_step<R, 1>(p, latent_dtype, lds, s);
    case 2: return launch_step<R, 2>(p, latent_dtype, lds, s);
    case 3: return launch_step<R, 3>(p, latent_dtype, lds, s);
    case 4: return launch_step<R, 4>(p, latent_dtype, lds, s);
    case 5: return launch_step<R, 5>(p, latent_dtype, lds, s);
    case 6: return launch_step<R, 6>(p, latent_dtype, lds, s);
    case 7: return launch_step<R, 7>(p, latent_dtype, lds, s);
    case 8: return launch_step<R, 8>(p, latent_dtype, lds, s);
    default: return hipErrorNotSupported;
  }
}

hipError_t wsvd_launch_step_float(wsvd_ctx* ctx, const wsvd_layer_desc& d, const void* x, const void* A_K, const void* A_V, const void* q,
                                  const void* q_scale, const void* B_K, const void* B_V, const wsvd_cache& cache, int max_seq_len,
                                  void* out, hipStream_t s) {
  if (!wsvd_step_deferred_float_ok(d)) return hipErrorNotSupported;
  FloatStepParams p = {};
  dim3 grid;
  int threads;
  wsvd_attn_plan(ctx, d, q, q_scale, B_K, B_V, cache, max_seq_len, out, p.a, grid, threads, 0);
  wsvd_append_params(ctx, d, x, nullptr, A_K, A_V, cache, p.ap);
  const int waves = d.rank == 64 ? 8 : 16;
  size_t lds = 0;
  if (d.latent_dtype == WSVD_BF16) {
    if (!wsvd_append_step_shape(ctx, d, waves, &p.helpers, &p.xs_stride, &lds) || lds > kStepLds) return hipErrorNotSupported;
    p.a.n_parts = p.helpers + 1;
  } else {
    p.a.n_parts = p.ap.ES;
  }
  p.n_proj = p.a.n_parts * 2 * d.n_kv_heads;
  if (ctx->opt.step_launches == 0 && !step_one_launch(ctx, d, p, waves, (int)(grid.x * grid.y * grid.z), max_seq_len)) return hipErrorNotSupported;
  // the words: behind those that the attention's own splits use, in the part of the workspace that is zero between launches
  const size_t plane = (size_t)d.batch * d.n_kv_heads * d.rank, words = (size_t)p.a.n_parts * 2 * plane;
  const size_t split = p.a.n_chunks > 1 ? (size_t)d.batch * d.n_q_heads * p.a.n_chunks * (d.rank + 2) : 0;
  if (split + words > wsvd_zero_words(d)) return hipErrorNotSupported;
  p.a.new_words = p.a.partials + split;
  p.ap.defer_words = p.a.new_words;
  p.a.new_ld = (long)d.n_kv_heads * d.rank;
  p.a.part_stride = (long)(2 * plane);
  if (p.a.timeline || p.ap.timeline) return hipErrorNotSupported;      // (profiling build: the stamps are the two launches')
  p.read = p.a.tickets;
  if (d.rank == 16) return launch_step_g<16>(p, d.latent_dtype, lds, s);
  if (d.rank == 32) return launch_step_g<32>(p, d.latent_dtype, lds, s);
  return launch_step_g<64>(p, d.latent_dtype, lds, s);
}
