// Decode attention over F32 / BF16 latent caches: the launches of its own, one work item per workgroup.
#include "wsvd_attn_generic_body.h"
#include "wsvd_internal.h"

template <int ESZ, int R, int G, bool NEWROW>
__global__ __launch_bounds__(256) void k_attn_generic(AttnParams p) {
  attn_generic_body<ESZ, R, G, NEWROW ? kRowPending : kNoRow>(p, p.seq_lens[blockIdx.z], blockIdx.x, blockIdx.y, blockIdx.z, NEWROW);
}

template <int ESZ, int R, bool NEWROW>
static hipError_t launch_gn(const AttnParams& p, dim3 grid, hipStream_t s) {
  switch (p.G) {
    case 1: hipLaunchKernelGGL((k_attn_generic<ESZ, R, 1, NEWROW>), grid, dim3(256), 0, s, p); break;
    case 2: hipLaunchKernelGGL((k_attn_generic<ESZ, R, 2, NEWROW>), grid, dim3(256), 0, s, p); break;
    case 3: hipLaunchKernelGGL((k_attn_generic<ESZ, R, 3, NEWROW>), grid, dim3(256), 0, s, p); break;
    case 4: hipLaunchKernelGGL((k_attn_generic<ESZ, R, 4, NEWROW>), grid, dim3(256), 0, s, p); break;
    case 5: hipLaunchKernelGGL((k_attn_generic<ESZ, R, 5, NEWROW>), grid, dim3(256), 0, s, p); break;
    case 6: hipLaunchKernelGGL((k_attn_generic<ESZ, R, 6, NEWROW>), grid, dim3(256), 0, s, p); break;
    case 7: hipLaunchKernelGGL((k_attn_generic<ESZ, R, 7, NEWROW>), grid, dim3(256), 0, s, p); break;
    case 8: hipLaunchKernelGGL((k_attn_generic<ESZ, R, 8, NEWROW>), grid, dim3(256), 0, s, p); break;
    default: return hipErrorNotSupported;
  }
  return hipGetLastError();
}
// p.pending set: the decode step's second launch, which finishes the rows (p.new_k, p.new_v, p.n_parts)
template <int ESZ, int R>
static hipError_t launch_g(const AttnParams& p, dim3 grid, hipStream_t s) {
  return p.pending ? launch_gn<ESZ, R, true>(p, grid, s) : launch_gn<ESZ, R, false>(p, grid, s);
}

hipError_t wsvd_launch_attn_generic(const AttnParams& p, int latent_dtype, int rank, dim3 grid, hipStream_t s) {
  if (latent_dtype == WSVD_F32) {
    if (rank == 16) return launch_g<4, 16>(p, grid, s);
    if (rank == 32) return launch_g<4, 32>(p, grid, s);
    if (rank == 64) return launch_g<4, 64>(p, grid, s);
  } else if (latent_dtype == WSVD_BF16) {
    if (rank == 16) return launch_g<2, 16>(p, grid, s);
    if (rank == 32) return launch_g<2, 32>(p, grid, s);
    if (rank == 64) return launch_g<2, 64>(p, grid, s);
  }
  return hipErrorInvalidValue;
}
