// Pressure forces on body surfaces (Sec. 2.3.1): the pointwise force
// dF_P = -P n dS (eq. Fpress) of every surface panel, its closed surface
// integral F_P (eq. FpressNet) per body, and the drag along the free stream
// with its coefficient 2 Drag / (rho |U|^2 A) (eq. CdP).
//
// The sums per body: segsum.h.
#include <cmath>

#include "../../include/pp.h"
#include "internal.h"
#include "segsum.h"

namespace pp {

namespace {
__global__ __launch_bounds__(kSumBlock) void k_forces(const double* __restrict__ p, const double* __restrict__ nx,
                                                       const double* __restrict__ ny, const double* __restrict__ ds,
                                                       ForceSegments segs, double ux, double uy, double rho,
                                                       double area, double* __restrict__ dfx,
                                                       double* __restrict__ dfy, pp_force* __restrict__ out) {
  sum_segment(segs, ux, uy, rho, area, out, [&](int64_t j, double& fx, double& fy) {
#pragma clang fp contract(off)
    const double pj = -p[j], dsj = ds[j];
    fx = (pj * nx[j]) * dsj;
    fy = (pj * ny[j]) * dsj;
    if (dfx) dfx[j] = fx;
    if (dfy) dfy[j] = fy;
  });
}
}  // namespace

void surface_forces(const double* p, const double* nx, const double* ny, const double* ds, int nseg,
                    const ForceSegments& seg, double ux, double uy, double rho, double area, double* dfx, double* dfy,
                    pp_force* out, hipStream_t s) {
  if (nseg <= 0) return;
  k_forces<<<(unsigned)(nseg * seg.slices), kSumBlock, 0, s>>>(p, nx, ny, ds, seg, ux, uy, rho, area, dfx, dfy, out);
}

}  // namespace pp
