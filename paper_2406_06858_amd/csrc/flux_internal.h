// Host-side declarations shared by the translation units of the library.
#pragma once
#include <hip/hip_runtime.h>
#include "flux.h"
#include "flux_device.h"

namespace flux {

// One entry per compiled tile configuration (index = public id - 1).
struct CfgInfo {
  int bm, bn, bk;
  int occupancy;   // workgroups per CU the kernel is built for
  int stages;      // slabs of B in LDS (more than two: the deep pipeline; the 256x256 tile holds one more of A)
  hipError_t (*launch[2])(int epi, int pro, int edge, int b_once, const GemmArgs& a, int grid, hipStream_t s);   // by layout of B: [K,N], [N,K]
};

constexpr int NUM_CFGS = 10;
extern CfgInfo g_cfgs[NUM_CFGS];

#define FLUX_DECLARE_CFG(ID) \
  hipError_t launch_cfg##ID##_nk0(int epi, int pro, int edge, int b_once, const GemmArgs& a, int grid, hipStream_t s); \
  hipError_t launch_cfg##ID##_nk1(int epi, int pro, int edge, int b_once, const GemmArgs& a, int grid, hipStream_t s);
FLUX_DECLARE_CFG(1)
FLUX_DECLARE_CFG(2)
FLUX_DECLARE_CFG(3)
FLUX_DECLARE_CFG(4)
FLUX_DECLARE_CFG(5)
FLUX_DECLARE_CFG(6)
FLUX_DECLARE_CFG(7)
FLUX_DECLARE_CFG(8)
FLUX_DECLARE_CFG(9)
FLUX_DECLARE_CFG(10)

}  // namespace flux
