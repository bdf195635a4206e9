// Marking of the lattice sites inside the cells for the interior viscosity
// (Sec. 1, Sec. 3.4): one work-group per cell runs inside::mark_cell, which
// states the ray-parity rule.  The marks are bytes in the site-ordered
// mask: bit k for a cell of viscosity class k (cells of different
// stiffness may carry different interior viscosities, Sec. 3.4), of which the
// lattice pass takes the highest (and clears the byte) to pick the relaxation
// time.  With one class every cell stores the same byte; with several the
// bits are joined atomically in one launch for all cells (a launch per class,
// plain stores, took 14.9 us each for 440 cells of two classes; this 22.5).
#include "interior_dev.h"

namespace hc {
namespace {

constexpr int kMarkThreads = 256;

__global__ __launch_bounds__(kMarkThreads) void k_mark_interior(Cells C, Mesh M, Lattice L,
                                                                unsigned char* __restrict__ mask,
                                                                const unsigned char* __restrict__ cls,
                                                                int* __restrict__ flags) {
  extern __shared__ float sp[];   // [nv][3] offsets
  __shared__ inside::Lds S;
  const int c = blockIdx.x, tid = threadIdx.x;
  const int64_t b3 = (int64_t)c * M.nv * 3;
  const int o[3] = {C.origin[3 * c], C.origin[3 * c + 1], C.origin[3 * c + 2]};
  inside::Grid G;
  for (int d = 0; d < 3; ++d) G.bc[d] = L.bc[d];
  G.n[0] = L.nx;
  G.n[1] = L.ny;
  G.n[2] = L.nz;
  G.le = L.le;
  G.le_delta = L.le_delta;
  const unsigned bit = 1u << (cls ? cls[c] : 0);
  auto mark = [&](int64_t h) {
    if (cls) atomicOr(reinterpret_cast<unsigned*>(mask) + (h >> 2), bit << (8 * (int)(h & 3)));
    else mask[h] = (unsigned char)bit;
  };
  inside::mark_cell(C.off + b3, sp, M.nv, M.tri, M.nt, o, G, [&](int x, int y, int z) { return site_of(L, x, y, z); },
                    mark, flags + 1, S, tid, kMarkThreads);
}

}  // namespace

hipError_t launch_mark_interior(const Cells& c, const Mesh& m, const Lattice& L, unsigned char* mask,
                                const unsigned char* cls, int* flags, hipStream_t s) {
  if (c.n == 0) return hipSuccess;
  const size_t lds = (size_t)m.nv * 3 * sizeof(float);
  hipLaunchKernelGGL(k_mark_interior, dim3(c.n), dim3(kMarkThreads), lds, s, c, m, L, mask, cls, flags);
  return hipGetLastError();
}

}  // namespace hc
