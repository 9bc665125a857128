// io.hip -- atoms between the caller's layout (n x dim, atom-id order) and the
// device's (double4 per atom, slot order): one copy of what the caller has, the
// rest made on the device.
#include <hip/hip_runtime.h>

#include "kernels.h"

namespace aqs {

namespace {

template <int D>
__global__ __launch_bounds__(kBlock) void k_load_atoms(Geom g, const double* pos, const uint8_t* types,
                                                       double4* pos4, int32_t* id, int32_t* inv) {
  const int i = blockIdx.x * kBlock + threadIdx.x;
  if (i >= g.n) return;
  pos4[g.atom_off + i] = make_double4(pos[(int64_t)i * D], pos[(int64_t)i * D + 1],
                                      D == 3 ? pos[(int64_t)i * D + 2] : 0.0, (double)types[i]);
  id[g.atom_off + i] = i;
  inv[g.atom_off + i] = i;
}

template <int D>
__global__ __launch_bounds__(kBlock) void k_pack_positions(Geom g, const double4* pos4, const int32_t* inv,
                                                           double* out) {
  const int i = blockIdx.x * kBlock + threadIdx.x;
  if (i >= g.n) return;
  const double4 p = pos4[g.atom_off + inv[g.atom_off + i]];
  out[(int64_t)i * D] = p.x;
  out[(int64_t)i * D + 1] = p.y;
  if (D == 3) out[(int64_t)i * D + 2] = p.z;
}

template <int D>
__global__ __launch_bounds__(kBlock) void k_pack_columns(Geom g, const double* x, const double* y, const double* z,
                                                         const int32_t* inv, double* out) {
  const int i = blockIdx.x * kBlock + threadIdx.x;
  if (i >= g.n) return;
  const int64_t gi = g.atom_off + inv[g.atom_off + i];
  out[(int64_t)i * D] = x[gi];
  out[(int64_t)i * D + 1] = y[gi];
  if (D == 3) out[(int64_t)i * D + 2] = z[gi];
}

}  // namespace

void launch_load_atoms(const Geom& g, int32_t dim, const double* pos, const uint8_t* types, double4* pos4,
                       int32_t* id, int32_t* inv, hipStream_t s) {
  if (dim == 3)
    hipLaunchKernelGGL(k_load_atoms<3>, dim3(g.nblocks), dim3(kBlock), 0, s, g, pos, types, pos4, id, inv);
  else
    hipLaunchKernelGGL(k_load_atoms<2>, dim3(g.nblocks), dim3(kBlock), 0, s, g, pos, types, pos4, id, inv);
}

void launch_pack_positions(const Geom& g, int32_t dim, const double4* pos4, const int32_t* inv, double* out,
                           hipStream_t s) {
  if (dim == 3)
    hipLaunchKernelGGL(k_pack_positions<3>, dim3(g.nblocks), dim3(kBlock), 0, s, g, pos4, inv, out);
  else
    hipLaunchKernelGGL(k_pack_positions<2>, dim3(g.nblocks), dim3(kBlock), 0, s, g, pos4, inv, out);
}

void launch_pack_columns(const Geom& g, int32_t dim, const double* x, const double* y, const double* z,
                         const int32_t* inv, double* out, hipStream_t s) {
  if (dim == 3)
    hipLaunchKernelGGL(k_pack_columns<3>, dim3(g.nblocks), dim3(kBlock), 0, s, g, x, y, z, inv, out);
  else
    hipLaunchKernelGGL(k_pack_columns<2>, dim3(g.nblocks), dim3(kBlock), 0, s, g, x, y, z, inv, out);
}

}  // namespace aqs
