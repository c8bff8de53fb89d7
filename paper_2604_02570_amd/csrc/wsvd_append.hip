// Latent append: c_K = x A_K[h], c_V = x A_V[h] for the new token of every sequence, rounded to the
// cache's storage format and written at row seq_lens[b] (decoding pipeline of Section 3.4).
//
// The factors arrive PACKED (wsvd_pack_factor_a): blocks of 32 latent channels x 16 model dims stored as the
// register image of a 32x32x16 matrix-core operand, so a wavefront's 64 x 16-byte load is one contiguous KiB
// and is the operand itself.
// The contraction over d_model is split into ES slices so that enough workgroups stream the factors;
// slice partials go to the workspace and the last workgroup of a (plane, kv head) to arrive sums them
// in slice order (deterministic), quantises and stores.  The very last workgroup bumps seq_lens.
//   bf16 factors and bf16 x: V_MFMA_F32_32X32X16_BF16, D[latent channel][sequence];
//   anything else (the all-fp32 configuration): vector ALU.
#include "wsvd_dev.h"
#include "wsvd_append_split.h"

template <int R, int FESZ, int DEFER = kNoDefer, int BB = kAppendBB>
__global__ __launch_bounds__(256) void k_append_valu(AppendParams p) { append_valu_body<R, FESZ, DEFER, BB>(p, (int)blockIdx.x); }

// ---------------------------------------------------------------- factor packing (set-up time)
__global__ __launch_bounds__(256) void k_pack_factor_a(const void* __restrict__ src, void* __restrict__ dst, int Hkv, int E, int R, int esz) {
  const int tiles = (R + 31) >> 5;
  const size_t total = (size_t)Hkv * tiles * 32 * E;       // packed elements, channels padded to a multiple of 32
  size_t i = (size_t)blockIdx.x * blockDim.x + threadIdx.x;
  if (i >= total) return;
  // decode the packed position
  const int e7 = (int)(i & 7); size_t r = i >> 3;
  const int c = (int)(r & 31); r >>= 5;
  const int g = (int)(r & 1); r >>= 1;
  const int eb = (int)(r % (size_t)(E >> 4)); r /= (size_t)(E >> 4);
  const int tile = (int)(r % tiles); const int kv = (int)(r / tiles);
  const int j = tile * 32 + c, e = eb * 16 + g * 8 + e7;
  const size_t sidx = ((size_t)kv * E + e) * R + j;
  if (esz == 4) ((uint32_t*)dst)[i] = j < R ? ((const uint32_t*)src)[sidx] : 0u;
  else ((uint16_t*)dst)[i] = j < R ? ((const uint16_t*)src)[sidx] : (uint16_t)0;
}

hipError_t wsvd_launch_pack_factor_a(const wsvd_layer_desc& d, const void* src, void* dst, hipStream_t s) {
  const size_t total = (size_t)d.n_kv_heads * ((d.rank + 31) / 32) * 32 * d.d_model;
  hipLaunchKernelGGL(k_pack_factor_a, dim3((unsigned)((total + 255) / 256)), dim3(256), 0, s, src, dst, d.n_kv_heads, d.d_model,
                     d.rank, d.factor_dtype == WSVD_F32 ? 4 : 2);
  return hipGetLastError();
}

template <int R, int NT, int DEFER = kNoDefer>
__global__ __launch_bounds__(NT) void k_append_split(AppendParams p, int SB, int xs_stride, int NP, unsigned long long* ll) {
  extern __shared__ __align__(16) uint8_t app_lds[];
  append_split_body<R, NT, DEFER>(p, SB, xs_stride, NP, ll, (int)blockIdx.x, (int)gridDim.x, (int)blockIdx.y, (int)gridDim.y, app_lds);
}

// sequences per workgroup: 16, or 32 for larger batches (all 32 columns of the matrix-core tile: half as many passes over
// the factors), fewer when the finisher's share of their hidden-state rows does not fit LDS
// helpers per unit: two for model dims from 1024 (one when the batch needs more than one group of 32 sequences: the
// finisher and one helper per unit and group are then one workgroup per CU for up to 64 sequences of 32 kv heads, a
// single round), none below (the "append_helpers" option overrides)
static int append_split_np(const wsvd_layer_desc& d, int opt_helpers = -1) {
  if (opt_helpers >= 0) return d.d_model >= 1024 ? opt_helpers : 0;
  return d.d_model >= 1024 ? (d.batch > 32 ? 1 : 2) : 0;
}
static int append_split_sb(const wsvd_layer_desc& d) {
  const int share = append_split_np(d) ? (d.d_model / 16 + 1) / 2 * 16 : d.d_model;
  int sb = d.batch > 16 ? 32 : 16;
  while (sb > 1 && (size_t)sb * (share + 8) * 2 > (size_t)144 * 1024) sb >>= 1;
  return sb;
}
static bool append_split_ok(const wsvd_layer_desc& d) {
  const int share = append_split_np(d) ? (d.d_model / 16 + 1) / 2 * 16 : d.d_model;
  return (size_t)append_split_sb(d) * (share + 8) * 2 <= (size_t)144 * 1024 && d.d_model % 16 == 0;
}
// 8-byte words the helpers push per launch (the workspace's append area holds them)
size_t wsvd_append_ll_words(const wsvd_layer_desc& d) {
  const int sb = append_split_sb(d);
  return (size_t)2 * d.n_kv_heads * ((d.batch + sb - 1) / sb) * 2 * sb * d.rank;
}

template <int R, int NT, int DEFER = kNoDefer>
static hipError_t launch_append_split(const AppendParams& p, const wsvd_layer_desc& d, int opt_helpers, unsigned long long* ll,
                                      hipStream_t s) {
  const int np = append_split_np(d, opt_helpers), sb = append_split_sb(d);
  const int share = np ? (d.d_model / 16 + 1) / 2 * 16 : d.d_model;
  const int stride = share + 8;                           // row stride = 4 dwords mod 32 banks: conflict-free operand reads
  const int groups = (d.batch + sb - 1) / sb;
  const int nw = NT / 64;
  size_t lds = (size_t)sb * stride * 2;
  const size_t red_bytes = (size_t)nw * sb * (R + 1) * 4;
  if (red_bytes > lds) lds = red_bytes;
  static LdsLimit limit;                                  // one per instantiation (the template makes it so)
  hipError_t e = wsvd_raise_lds(limit, (const void*)k_append_split<R, NT, DEFER>, 150 * 1024);
  if (e != hipSuccess) return e;
  dim3 grid((unsigned)(2 * d.n_kv_heads * (np + 1)), (unsigned)groups);
  hipLaunchKernelGGL((k_append_split<R, NT, DEFER>), grid, dim3(NT), lds, s, p, sb, stride, np, ll);
  return hipGetLastError();
}

static bool append_mfma_path(const wsvd_layer_desc& d);
int wsvd_step_slices(const wsvd_ctx* ctx, const wsvd_layer_desc& d);
// The decode step's projection launch: `ns` equal d_model slices per (plane, kv head), partial sums to p.defer_out.
static void project_shape(const wsvd_layer_desc& d, int ns, int nw, int* sb, int* stride, int* groups, size_t* lds) {
  const int nks = d.d_model / 16;
  const int share = (nks + ns - 1) / ns * 16;
  *stride = share + 8;
  *sb = 16;
  while (*sb > 1 && (size_t)*sb * *stride * 2 > (size_t)144 * 1024) *sb >>= 1;
  *groups = (d.batch + *sb - 1) / *sb;
  const size_t xs = (size_t)*sb * *stride * 2, red = (size_t)nw * *sb * (d.rank + 1) * 4;
  *lds = xs > red ? xs : red;
}
void wsvd_append_project_shape(const wsvd_ctx* ctx, const wsvd_layer_desc& d, int waves, int* slices, int* sb, int* stride, int* groups, size_t* lds) {
  *slices = wsvd_step_slices(ctx, d);
  project_shape(d, *slices, waves, sb, stride, groups, lds);
}
template <int R, int NT>
static hipError_t launch_append_project(const AppendParams& p, const wsvd_layer_desc& d, int ns, hipStream_t s) {
  int sb, stride, groups;
  size_t lds;
  project_shape(d, ns, NT / 64, &sb, &stride, &groups, &lds);
  if (lds > (size_t)150 * 1024) return hipErrorInvalidValue;
  static LdsLimit limit;
  hipError_t e = wsvd_raise_lds(limit, (const void*)k_append_split<R, NT, kDeferSlices>, 150 * 1024);
  if (e != hipSuccess) return e;
  dim3 grid((unsigned)(2 * d.n_kv_heads * ns), (unsigned)groups);
  hipLaunchKernelGGL((k_append_split<R, NT, kDeferSlices>), grid, dim3(NT), lds, s, p, sb, stride, ns, (unsigned long long*)nullptr);
  return hipGetLastError();
}

// The same projection as part of the one-launch step: one group of all sequences.
bool wsvd_append_step_shape(const wsvd_ctx* ctx, const wsvd_layer_desc& d, int waves, int* helpers, int* xs_stride, size_t* lds) {
  if (d.batch > append_split_sb(d)) return false;
  *helpers = append_split_np(d, ctx->opt.append_helpers);
  *xs_stride = (*helpers ? (d.d_model / 16 + 1) / 2 * 16 : d.d_model) + 8;
  const size_t xs = (size_t)d.batch * *xs_stride * 2, red = (size_t)waves * d.batch * (d.rank + 1) * 4;
  *lds = xs > red ? xs : red;
  return true;
}

template <int R>
static hipError_t launch_append_valu_defer(const AppendParams& p, hipStream_t s) {
  const dim3 grid((unsigned)(p.ES * p.Hkv * 2));
  if (p.B == 1) hipLaunchKernelGGL((k_append_valu<R, 4, kDeferShares, 1>), grid, dim3(256), 0, s, p);
  else hipLaunchKernelGGL((k_append_valu<R, 4, kDeferShares>), grid, dim3(256), 0, s, p);
  return hipGetLastError();
}

// slices of the decode step's projection launch: about one workgroup per CU, at most 4, slices of whole k-steps
int wsvd_step_slices(const wsvd_ctx* ctx, const wsvd_layer_desc& d) {
  int ns = ctx->opt.step_slices > 0 ? ctx->opt.step_slices : ctx->n_cu / (2 * d.n_kv_heads);
  if (ns > 4) ns = 4;
  while (ns > 1 && d.d_model / 16 / ns < 4) ns--;
  return ns < 1 ? 1 : ns;
}
bool wsvd_step_deferred_ok(const wsvd_layer_desc& d) {
  return append_mfma_path(d) && d.latent_dtype == WSVD_I8 && (d.rank == 32 || d.rank == 64) &&
         d.n_q_heads / d.n_kv_heads <= 4 && d.d_model % 16 == 0 && d.batch <= kAppendMaxB;
}
// fp32 and bf16 latents (x and factors of the same type): the vector-ALU attention finishes the row.  The partial sums are
// the append's own (its slices in fp32, its shares in bf16), so rows and outputs are those of the two calls bit for bit.
bool wsvd_step_deferred_float_ok(const wsvd_layer_desc& d) {
  const bool f32 = d.latent_dtype == WSVD_F32, bf16 = d.latent_dtype == WSVD_BF16 && append_split_ok(d);
  return (f32 || bf16) && d.rank <= 64 && d.batch <= kAppendMaxB && d.d_model % 64 == 0;
}
// where the step's partial sums and its pending words live: inside the sliced kernels' partial area of the workspace
bool wsvd_step_partials(const wsvd_ctx* ctx, const wsvd_layer_desc& d, float** parts, int** pending, int* n_parts) {
  AppendParams p;
  wsvd_cache none = {};
  wsvd_append_params(ctx, d, nullptr, nullptr, nullptr, nullptr, none, p);
  const int ns = d.latent_dtype == WSVD_F32 ? p.ES : d.latent_dtype == WSVD_BF16 ? append_split_np(d, ctx->opt.append_helpers) + 1
                                                                                 : wsvd_step_slices(ctx, d);
  const size_t part_floats = (size_t)ns * 2 * d.batch * d.n_kv_heads * d.rank;
  if (part_floats > (size_t)2 * d.n_kv_heads * (d.d_model / 64) * d.batch * d.rank) return false;
  *parts = p.partials; *pending = (int*)(p.partials + part_floats); *n_parts = ns;
  return true;
}
hipError_t wsvd_launch_append_project(const wsvd_ctx* ctx, const wsvd_layer_desc& d, const void* x, const void* A_K,
                                      const void* A_V, const wsvd_cache& cache, float** parts, int** pending, int* n_parts,
                                      hipStream_t s) {
  AppendParams p;
  wsvd_append_params(ctx, d, x, nullptr, A_K, A_V, cache, p);
  int ns = 0;
  if (!wsvd_step_partials(ctx, d, parts, pending, &ns)) return hipErrorNotSupported;
  p.defer_out = *parts;
  p.pending = *pending;
  if (ctx->opt.timeline_kernel != 1) p.timeline = nullptr;    // (profiling build: by default a step's stamps are its attention launch's)
  *n_parts = ns;
  if (d.latent_dtype == WSVD_F32) {
    switch (d.rank) {
      case 16: return launch_append_valu_defer<16>(p, s);
      case 32: return launch_append_valu_defer<32>(p, s);
      case 64: return launch_append_valu_defer<64>(p, s);
      default: return hipErrorNotSupported;
    }
  }
  if (d.latent_dtype == WSVD_BF16) {
    switch (d.rank) {
      case 16: return launch_append_split<16, 1024, kDeferShares>(p, d, ctx->opt.append_helpers, nullptr, s);
      case 32: return launch_append_split<32, 1024, kDeferShares>(p, d, ctx->opt.append_helpers, nullptr, s);
      case 64: return launch_append_split<64, 512, kDeferShares>(p, d, ctx->opt.append_helpers, nullptr, s);
      default: return hipErrorNotSupported;
    }
  }
  switch (d.rank) {
    case 32: return launch_append_project<32, 512>(p, d, ns, s);      // (8 waves: 6.7 us at config 3; 16: 6.9 us; 4: 7.4 us)
    case 64: return launch_append_project<64, 512>(p, d, ns, s);
    default: return hipErrorNotSupported;
  }
}

// d_model slices per (plane, kv head).
// One CU cannot pull more than a few tens of GB/s on its own, so the factor stream has to be spread over all of
// them: the MFMA path aims at about one workgroup per CU (256) and merges the slices through the ticket.
// The vector-ALU path keeps slices of at most 256 elements (its LDS staging size).
static bool append_mfma_path(const wsvd_layer_desc& d) { return d.factor_dtype == WSVD_BF16 && d.x_dtype == WSVD_BF16; }
int wsvd_append_esplits(const wsvd_ctx* ctx, const wsvd_layer_desc& d) {
  if (!append_mfma_path(d)) {
    int esl = kAppendMaxESL;
    while (esl > 64 && d.d_model % esl != 0) esl >>= 1;
    return d.d_model / esl;
  }
  const int units = d.d_model / 64;                              // slices are multiples of 64 elements
  int want = ctx->opt.append_mode > 0 ? ctx->opt.append_mode : 256 / (2 * d.n_kv_heads);
  if (want < 1) want = 1;
  // smallest slice count >= want whose slices fit the kernel's LDS staging; else the largest count that exists
  int es = units;
  for (int c = 1; c <= units; c++) {
    if (units % c != 0 || d.d_model / c > kAppendMfmaESL) continue;
    es = c;
    if (c >= want) break;
  }
  return es;
}
static size_t wsvd_append_pushed_floats(const wsvd_layer_desc& d) {
  return append_mfma_path(d) && append_split_ok(d) ? (2 * wsvd_append_ll_words(d) + 3) / 4 * 4 : 0;
}
size_t wsvd_zero_words(const wsvd_layer_desc& d) {
  return ((wsvd_attn_partial_floats(d) + 3) / 4 * 4 + wsvd_append_pushed_floats(d)) / 2;
}
size_t wsvd_append_partial_floats(const wsvd_layer_desc& d) {
  // the pushed words of the default kernel (which are zero between launches), then the sliced kernels' partial sums
  // (the most slices an option can ask for)
  // (+ one word per sequence behind the decode step's partial sums, which use this area too)
  const size_t sliced = (size_t)2 * d.n_kv_heads * (d.d_model / 64) * d.batch * d.rank + ((size_t)d.batch + 3) / 4 * 4;
  return wsvd_append_pushed_floats(d) + sliced;
}

void wsvd_append_params(const wsvd_ctx* ctx, const wsvd_layer_desc& d, const void* x, const void* x_scale, const void* A_K,
                        const void* A_V, const wsvd_cache& cache, AppendParams& p) {
  p = AppendParams{};
  p.x = x; p.x_scale = (const uint16_t*)x_scale;
  p.A[0] = A_K; p.A[1] = A_V;
  p.codes[0] = (uint8_t*)cache.k_codes; p.codes[1] = (uint8_t*)cache.v_codes;
  p.meta[0] = (uint16_t*)cache.k_meta; p.meta[1] = (uint16_t*)cache.v_meta;
  p.seq_lens = cache.seq_lens;
  p.tickets = (int*)ctx->ws + kWsCounterInts / 2;
  p.partials = (float*)((char*)ctx->ws + (size_t)kWsCounterInts * 4) + (wsvd_attn_partial_floats(d) + 3) / 4 * 4 + wsvd_append_pushed_floats(d);
  p.err_word = ctx->err_word;
  p.B = d.batch; p.E = d.d_model; p.Hkv = d.n_kv_heads; p.t_cap = d.t_cap;
  p.ES = wsvd_append_esplits(ctx, d); p.ESL = d.d_model / p.ES;
  p.x_dtype = d.x_dtype; p.factor_dtype = d.factor_dtype; p.latent_dtype = d.latent_dtype;
  p.one_seq = -1;
  p.timeline = ctx->timeline_bytes >= (size_t)4096 * kTimelineWaves * kTimelineSlots * sizeof(long long) ? ctx->timeline : nullptr;
}

// waves per workgroup of the MFMA path: each wave gets a multiple of 16 elements, at least 64; up to 16 waves
// (rank 64: 8, register budget)
int wsvd_append_mfma_waves(const wsvd_ctx* ctx, const wsvd_layer_desc& d) {
  const int esl = d.d_model / wsvd_append_esplits(ctx, d);
  int nw = d.rank == 64 ? 8 : 16;
  while (nw > 4 && ((esl / nw) % 16 != 0 || esl / nw < 64)) nw >>= 1;
  return nw;
}
bool wsvd_append_uses_mfma(const wsvd_layer_desc& d) { return append_mfma_path(d); }

hipError_t wsvd_launch_append(const wsvd_ctx* ctx, const wsvd_layer_desc& d, const void* x, const void* x_scale,
                              const void* A_K, const void* A_V, const wsvd_cache& cache, hipStream_t s, int one_seq,
                              const wsvd_paged_cache* paged) {
  if (paged && !(d.rank <= 64 && append_mfma_path(d) && ctx->opt.append_mode == 0 && append_split_ok(d) &&
                 (d.latent_dtype == WSVD_I8 || d.latent_dtype == WSVD_I4)))
    return hipErrorNotSupported;           // paged cache: quantised latents through the default kernel
  if (d.rank > 64) {
    // ranks 96 / 128 (int8 latents, bf16 hidden states and factors): the tiled projection with one token per sequence,
    // then its length update: two launches
    if (one_seq >= 0) return hipErrorNotSupported;
    return wsvd_launch_prefill_project(ctx, d, x, 1, -1, A_K, A_V, cache, s);
  }
  AppendParams p;
  wsvd_append_params(ctx, d, x, x_scale, A_K, A_V, cache, p);
  p.one_seq = one_seq;
  if (paged) { p.block_table = paged->block_table; p.page_rows = paged->page_rows; p.max_pages = paged->max_pages; p.n_pages = paged->n_pages; }
  if (d.d_model % 64 != 0 || d.batch > kAppendMaxB) return hipErrorInvalidValue;
  dim3 grid((unsigned)(p.ES * p.Hkv * 2));
  const bool f32 = d.factor_dtype == WSVD_F32;
  if (append_mfma_path(d) && ctx->opt.append_mode == 0 && append_split_ok(d)) {
    // the default ("append_mode" n > 0 asks for the kernel with n equal slices merged by the last arriver instead)
    unsigned long long* ll = (unsigned long long*)((char*)ctx->ws + (size_t)kWsCounterInts * 4 + (wsvd_attn_partial_floats(d) + 3) / 4 * 16);
    switch (d.rank) {
      case 16: return launch_append_split<16, 1024>(p, d, ctx->opt.append_helpers, ll, s);
      case 32: return launch_append_split<32, 1024>(p, d, ctx->opt.append_helpers, ll, s);
      case 64: return launch_append_split<64, 512>(p, d, ctx->opt.append_helpers, ll, s);
      default: return hipErrorInvalidValue;
    }
  }
  if (append_mfma_path(d)) {
    int nw = wsvd_append_mfma_waves(ctx, d);
    if (d.batch > 32) {
      // two groups of 32 sequences per pass over the factors; the second set of accumulators needs the register
      // budget of a workgroup of at most 8 waves
      if (nw > 8) nw = 8;
      dim3 block((unsigned)(nw * 64));
      switch (d.rank) {
        case 16: hipLaunchKernelGGL((k_append_mfma<16, 512, 2>), grid, block, 0, s, p); break;
        case 32: hipLaunchKernelGGL((k_append_mfma<32, 512, 2>), grid, block, 0, s, p); break;
        case 64: hipLaunchKernelGGL((k_append_mfma<64, 512, 2>), grid, block, 0, s, p); break;
        default: return hipErrorInvalidValue;
      }
      return hipGetLastError();
    }
    dim3 block((unsigned)(nw * 64));
    switch (d.rank) {
      case 16: hipLaunchKernelGGL((k_append_mfma<16, 1024, 1>), grid, block, 0, s, p); break;
      case 32: hipLaunchKernelGGL((k_append_mfma<32, 1024, 1>), grid, block, 0, s, p); break;
      case 64: hipLaunchKernelGGL((k_append_mfma<64, 512, 1>), grid, block, 0, s, p); break;
      default: return hipErrorInvalidValue;
    }
    return hipGetLastError();
  }
  dim3 block(256);
  switch (d.rank) {
    case 16: if (f32) hipLaunchKernelGGL((k_append_valu<16, 4>), grid, block, 0, s, p); else hipLaunchKernelGGL((k_append_valu<16, 2>), grid, block, 0, s, p); break;
    case 32: if (f32) hipLaunchKernelGGL((k_append_valu<32, 4>), grid, block, 0, s, p); else hipLaunchKernelGGL((k_append_valu<32, 2>), grid, block, 0, s, p); break;
    case 64: if (f32) hipLaunchKernelGGL((k_append_valu<64, 4>), grid, block, 0, s, p); else hipLaunchKernelGGL((k_append_valu<64, 2>), grid, block, 0, s, p); break;
    default: return hipErrorInvalidValue;
  }
  return hipGetLastError();
}

// ---------------------------------------------------------------- store of latents computed elsewhere
// The quantise-and-store half of the append for callers that produce the latents with another GEMM (the
// int4-weight / int8-activation projection of the quantised setting, Section 4.2).  One workgroup per sequence:
// it reads the sequence's length once, stores the 2*Hkv rows with R lanes per row and then advances the length,
// so no cross-workgroup ordering is needed.
template <int R>
__global__ __launch_bounds__(1024) void k_latent_store(AppendParams p, const float* __restrict__ cK,
                                                       const float* __restrict__ cV, long ld) {
  const int b = blockIdx.x;
  const int total = 2 * p.Hkv * R;     // a multiple of 64 whenever the latents are quantised (R >= 32)
  // every thread reads the length itself (one broadcast load) together with its first kAhead latents: one round trip for
  // up to 4096 latents a sequence (two of them, 32 heads of rank 32, took a second trip: 6.0 -> 5.4 us)
  constexpr int kAhead = 4;
  const int n = __hip_atomic_load(p.seq_lens + b, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT);
  auto latent = [&](int i) {
    const int row = i / R;
    return (row >= p.Hkv ? cV + (size_t)(row - p.Hkv) * R : cK + (size_t)row * R)[(size_t)b * ld + i % R];
  };
  float ahead[kAhead];
#pragma unroll
  for (int k = 0; k < kAhead; k++)
    if (k == 0 || k * (int)blockDim.x < total) ahead[k] = latent(min((int)(threadIdx.x + k * blockDim.x), total - 1));   // (uniform)
  if (n < 0 || n >= p.t_cap) {
    if (threadIdx.x == 0) atomicExch(p.err_word, (int)WSVD_E_CAPACITY);
    return;
  }
  auto store = [&](int idx, float c) {
    const int row = idx / R, pl = row >= p.Hkv ? 1 : 0;
    store_row_lanes<R>(p, pl, b, row - pl * p.Hkv, n, idx % R, c);
  };
#pragma unroll
  for (int k = 0; k < kAhead; k++) {
    const int idx = threadIdx.x + k * blockDim.x;
    if (idx < total) store(idx, ahead[k]);
  }
  for (int idx = threadIdx.x + kAhead * blockDim.x; idx < total; idx += blockDim.x) store(idx, latent(idx));
  __syncthreads();     // every thread has consumed the old length
  if (threadIdx.x == 0) p.seq_lens[b] = n + 1;
}

hipError_t wsvd_launch_latent_store(const wsvd_ctx* ctx, const wsvd_layer_desc& d, const float* cK, const float* cV,
                                    int64_t ld, const wsvd_cache& cache, hipStream_t s) {
  AppendParams p = {};
  p.codes[0] = (uint8_t*)cache.k_codes; p.codes[1] = (uint8_t*)cache.v_codes;
  p.meta[0] = (uint16_t*)cache.k_meta; p.meta[1] = (uint16_t*)cache.v_meta;
  p.seq_lens = cache.seq_lens;
  p.err_word = ctx->err_word;
  p.B = d.batch; p.E = d.d_model; p.Hkv = d.n_kv_heads; p.t_cap = d.t_cap;
  p.latent_dtype = d.latent_dtype;
  const int total = 2 * d.n_kv_heads * d.rank;
  int threads = (total + 63) / 64 * 64;
  if (threads > 1024) threads = 1024;
  dim3 grid((unsigned)d.batch), block((unsigned)threads);
  switch (d.rank) {
    case 16: hipLaunchKernelGGL((k_latent_store<16>), grid, block, 0, s, p, cK, cV, (long)ld); break;
    case 32: hipLaunchKernelGGL((k_latent_store<32>), grid, block, 0, s, p, cK, cV, (long)ld); break;
    case 64: hipLaunchKernelGGL((k_latent_store<64>), grid, block, 0, s, p, cK, cV, (long)ld); break;
    default: return hipErrorInvalidValue;
  }
  return hipGetLastError();
}
