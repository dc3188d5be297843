// Launches of the small-grid stage tiles (wiu_stage.hpp), gfx950.
#include "wiu_stage.hpp"

namespace wiu {

// Tiles of 8 x 8 nodes.  While every tile can have a compute unit of its own a
// workgroup takes 384 lanes (352 side fluxes of 5-2MP in one round, the nodal
// fluxes in a short second one: the shortest stage); beyond that 256, four
// workgroups a unit, so that one's loads run beside another's fluxes.  RK3
// steps of 5-2MP, microseconds with 384 / 256 lanes: 27.5 / 29.8 on 67 x 59
// nodes, 33.5 / 35.2 on 131 x 123, 49.2 / 39.1 on 195 x 187.  Tiles of 16 x 8
// by 512 lanes: 31.8, 32.8, 52.7.
constexpr int ST_X = 8, ST_Y = 8, ST_UNITS = 256;

template <int SC, int NT, bool OPT, bool PPM>
__global__ void __launch_bounds__(NT) stage_kernel(StageArgs a) {
  __shared__ StageLds<SC, ST_X, ST_Y, OPT> lds;
  const int ntx = (a.s.d.nx + ST_X - 1) / ST_X;
  const int lid = xcd_remap(blockIdx.x, gridDim.x);
  stage_tile<SC, ST_X, ST_Y, NT, OPT, PPM>(a, lid % ntx, lid / ntx, lid, gridDim.x, lds);
}

template <int SC, bool OPT, bool PPM> void launch_stage_o(const StageArgs& a, hipStream_t st) {
  const Dims& d = a.s.d;
  const int tiles = ((d.nx + ST_X - 1) / ST_X) * ((d.ny + ST_Y - 1) / ST_Y);
  if (tiles <= ST_UNITS)
    hipLaunchKernelGGL((stage_kernel<SC, 384, OPT, PPM>), dim3(tiles), dim3(384), 0, st, a);
  else
    hipLaunchKernelGGL((stage_kernel<SC, 256, OPT, PPM>), dim3(tiles), dim3(256), 0, st, a);
}

template <int SC> hipError_t launch_stage_s(const StageArgs& a, hipStream_t st) {
  if (a.s.vars != 0 || a.s.ah != 1.0 || a.s.weights != 0 || a.s.split != 0)
    launch_stage_o<SC, true, true>(a, st);
  else if (a.s.ppm)
    launch_stage_o<SC, false, true>(a, st);
  else
    launch_stage_o<SC, false, false>(a, st);
  return hipGetLastError();
}

hipError_t launch_stage(int scheme, const StageArgs& a, hipStream_t st) {
  switch (scheme) {
    case 0: return launch_stage_s<0>(a, st);
    case 1: return launch_stage_s<1>(a, st);
    case 2: return launch_stage_s<2>(a, st);
    case 3: return launch_stage_s<3>(a, st);
    case 4: return launch_stage_s<4>(a, st);
    case 5: return launch_stage_s<5>(a, st);
    case 6: return launch_stage_s<6>(a, st);
    case 7: return launch_stage_s<7>(a, st);
    default: return hipErrorInvalidValue;
  }
}

// Grids of at most 65536 nodes step with the stage tiles, larger ones with the sweeps.
// RK3 steps with stage tiles / sweeps, microseconds: 5-2MP 27.5 / 53.1 on 67 x 59
// nodes, 39.1 / 60.4 on 195 x 187, 60.9 / 65.4 on 259 x 251, 105 / 88 on 387 x 379;
// 7-4MP 83 / 85 and 3-1MP 50 / 59 on 259 x 251.  Below the line the sweeps' time is
// the latency of their launches, above it the tiles pay for their halos.  Beyond
// 1400 tiles (65536 nodes fill 1024) lines that leave the tiles' last row or column
// empty count: 7281 x 9, 1822 tiles, 94.4 / 88.5, 7-6MP 141 / 120, but 5000 x 13, 1250
// tiles, 73.5 / 78.3 and 101 / 97.  On grids of a few rows or columns the sweep
// across them is as empty: 32768 x 2, 4096 tiles, 174 / 189 and 239 / 236, 3 x 20000
// 152 / 279; 65536 x 1 300 / 312, but 7-6MP, whose tiles' halo is nearly twice as wide,
// 420 / 355, 24576 x 1 173 / 163 and 8192 x 1, 1024 tiles, 82 / 93.
bool use_stage_tiles(int scheme, int nx, int ny) {
  if ((long long)nx * ny > 65536) return false;
  const int tiles = ((nx + ST_X - 1) / ST_X) * ((ny + ST_Y - 1) / ST_Y);
  if (ny == 1 && scheme >= 4) return tiles <= 1024;
  return tiles <= 1400 || ny <= ST_Y || nx <= 3 * ST_X;
}

}  // namespace wiu
