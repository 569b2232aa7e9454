// Instantiates the GEMM kernel family for ONE tile configuration and layout of B; compiled once for each
// with -DFLUX_CFG_ID=<id> -DFLUX_B_NK=<0|1> so that they build in parallel.
#include "flux_internal.h"

namespace flux {

#if FLUX_CFG_ID == 1
#define FLUX_CFG_PARAMS 256, 256, 64, 2, 2, 3, 2, 1   // 128x128 per wave, one workgroup per CU
#elif FLUX_CFG_ID == 2
#define FLUX_CFG_PARAMS 256, 128, 64, 2, 2, 3, 3, 1   // 128x64 per wave: twice the tiles of 256x256; three LDS stages
#elif FLUX_CFG_ID == 3
#define FLUX_CFG_PARAMS 128, 128, 64, 2, 2, 2, 2, 2   // 64x64 per wave
#elif FLUX_CFG_ID == 4
#define FLUX_CFG_PARAMS 64, 64, 64, 2, 2, 2, 2, 2     // 32x32 per wave, small problems
#elif FLUX_CFG_ID == 5
#define FLUX_CFG_PARAMS 64, 128, 64, 2, 2, 2, 2, 2    // decode, M <= 64
#elif FLUX_CFG_ID == 6
#define FLUX_CFG_PARAMS 32, 128, 64, 1, 4, 2, 2, 2    // decode, M <= 32
#elif FLUX_CFG_ID == 7
#define FLUX_CFG_PARAMS 64, 64, 64, 2, 2, 6, 6, 1     // decode, M <= 64: six LDS stages, one workgroup per CU
#elif FLUX_CFG_ID == 8
#define FLUX_CFG_PARAMS 32, 128, 64, 1, 4, 6, 6, 1    // decode, M <= 32: six LDS stages
#elif FLUX_CFG_ID == 9
#define FLUX_CFG_PARAMS 64, 128, 64, 2, 2, 4, 4, 1    // M <= 256: four LDS stages
#elif FLUX_CFG_ID == 10
#define FLUX_CFG_PARAMS 64, 128, 64, 2, 2, 3, 3, 2    // few rows over a long K: 64x128, three stages, two workgroups per CU
#else
#error "FLUX_CFG_ID must be 1..10"
#endif
typedef TileCfg<FLUX_CFG_PARAMS, FLUX_B_NK> Cfg;     // B as [K,N] / [N,K]

// Tiles that few rows over large weights take have a second set of kernels, which stream B.
constexpr bool MAYBE_ONCE = FLUX_CFG_ID == 2 || FLUX_CFG_ID == 7 || FLUX_CFG_ID == 8 || FLUX_CFG_ID == 9;

template <int EPI, int PRO, bool B_ONCE, int PARTIALS>
static hipError_t launch_two(int edge, const GemmArgs& a, int grid, hipStream_t s) {
  if (edge) hipLaunchKernelGGL((gemm_kernel_dma<Cfg, EPI, PRO, true, B_ONCE, PARTIALS>), dim3(grid), dim3(Cfg::NT), 0, s, a);
  else hipLaunchKernelGGL((gemm_kernel_dma<Cfg, EPI, PRO, false, B_ONCE, PARTIALS>), dim3(grid), dim3(Cfg::NT), 0, s, a);
  return hipGetLastError();
}

template <int PARTIALS>
static hipError_t launch_resident(const GemmArgs& a, int grid, hipStream_t s) {
  if (a.R <= 4) hipLaunchKernelGGL((gemm_kernel_dma_resident<Cfg, 3, PARTIALS>), dim3(grid), dim3(Cfg::NT), 0, s, a);
  else hipLaunchKernelGGL((gemm_kernel_dma_resident<Cfg, FLUX_MAX_RANKS - 1, PARTIALS>), dim3(grid), dim3(Cfg::NT), 0, s, a);
  return hipGetLastError();
}

// `edge`: the tile does not divide the shape (masked loads and stores).
template <int EPI, int PRO>
static hipError_t launch_one(int edge, int b_once, const GemmArgs& a, int grid, hipStream_t s) {
  if constexpr (EPI == EPI_RS && Cfg::NB == 2 && Cfg::OCC == 1) {
    if (a.persist_blocks > 0) {          // (only planned for shapes the tile divides)
      if (a.partial_f32) return launch_resident<1>(a, grid, s);
      return launch_resident<0>(a, grid, s);
    }
  }
  if constexpr (EPI == EPI_RS && Cfg::BM * Cfg::BN >= 256 * 256) {          // (see gemm_tail)
    return a.partial_f32 ? launch_two<EPI, PRO, false, 1>(edge, a, grid, s) : launch_two<EPI, PRO, false, 0>(edge, a, grid, s);
  } else {
    if constexpr (MAYBE_ONCE && (EPI == EPI_RS || PRO == PRO_CHUNKS))
      if (b_once) return launch_two<EPI, PRO, true, -1>(edge, a, grid, s);
    return launch_two<EPI, PRO, false, -1>(edge, a, grid, s);
  }
}

#define FLUX_CAT2(a, b, c, d) a##b##c##d
#define FLUX_CAT(a, b, c, d) FLUX_CAT2(a, b, c, d)

hipError_t FLUX_CAT(launch_cfg, FLUX_CFG_ID, _nk, FLUX_B_NK)(int epi, int pro, int edge, int b_once, const GemmArgs& a, int grid, hipStream_t s) {
  if (epi == EPI_RS) return launch_one<EPI_RS, PRO_NONE>(edge, b_once, a, grid, s);
  if (pro == PRO_WAIT) return launch_one<EPI_PLAIN, PRO_WAIT>(edge, b_once, a, grid, s);
  if (pro == PRO_CHUNKS) return launch_one<EPI_PLAIN, PRO_CHUNKS>(edge, b_once, a, grid, s);
  return launch_one<EPI_PLAIN, PRO_NONE>(edge, b_once, a, grid, s);
}

}  // namespace flux
