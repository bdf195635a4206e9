// Marking of the lattice sites inside the cells for the interior viscosity
// (Sec. 1, Sec. 3.4): one work-group per cell runs inside::mark_cell, which
// states the ray-parity rule.  The marks are bytes in the site-ordered
// mask: bit k for a cell of viscosity class k (cells of different
// stiffness may carry different interior viscosities, Sec. 3.4), of which the
// lattice pass takes the highest (and clears the byte) to pick the relaxation
// time.  Cells of one class store plain bytes.  Several classes, whose marks
// may share a byte, are marked by one launch that joins the bits atomically
// (one 32-bit atomic per site), or by one launch of plain stores per class in
// increasing order; see kCellsPerClass.
#include "interior_dev.h"

namespace hc {
namespace {

constexpr int kMarkThreads = 256;

// From this many cells per class on, a launch per class.  It costs about 15 us
// a class (latency) and then only the stores; the atomics cost 26 ns a cell
// whatever the classes, the stores 10 to 19.  Atomic and per-class launches in
// us, every other cell of two classes: 24 and 33 at 440 cells, 47 and 44 at
// 1160, 78 and 69 at 2320, 485 and 388 at 18,600; four classes drawn at
// random: 75 and 83 at 2320, 138 and 98 at 4650; eight: 137 and 162 at 4650,
// 253 and 210 at 9300.
constexpr int kCellsPerClass = 640;

// JOIN: atomically, whatever the cell's class; else plain stores for the cells
// of one class (only_class, or all of them when negative).
template <bool JOIN>
__global__ __launch_bounds__(kMarkThreads) void k_mark_interior(Cells C, Mesh M, Lattice L,
                                                                unsigned char* __restrict__ mask,
                                                                const unsigned char* __restrict__ cls,
                                                                int only_class, int* __restrict__ flags) {
  extern __shared__ float sp[];   // [nv][3] offsets
  __shared__ inside::Lds S;
  const int c = blockIdx.x, tid = threadIdx.x;
  if (!JOIN && only_class >= 0 && cls[c] != only_class) return;   // another class's launch
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
    if (JOIN) atomicOr(reinterpret_cast<unsigned*>(mask) + (h >> 2), bit << (8 * (int)(h & 3)));
    else mask[h] = (unsigned char)bit;
  };
  inside::mark_cell(C.off + b3, sp, M.nv, M.tri, M.nt, o, G, [&](int x, int y, int z) { return site_of(L, x, y, z); },
                    mark, flags + 1, S, tid, kMarkThreads);
}

}  // namespace

hipError_t launch_mark_interior(const Cells& c, const Mesh& m, const Lattice& L, unsigned char* mask,
                                const unsigned char* cls, int n_class, int* flags, hipStream_t s) {
  if (c.n == 0) return hipSuccess;
  const size_t lds = (size_t)m.nv * 3 * sizeof(float);
  auto go = [&](auto kern, int only_class) {
    hipLaunchKernelGGL(kern, dim3(c.n), dim3(kMarkThreads), lds, s, c, m, L, mask, cls, only_class, flags);
    return hipGetLastError();
  };
  if (!cls) return go(k_mark_interior<false>, -1);
  if (c.n < kCellsPerClass * n_class) return go(k_mark_interior<true>, -1);
  // in increasing order, so that the highest class of a site is stored last
  for (int k = 0; k < n_class; ++k) {
    const hipError_t e = go(k_mark_interior<false>, k);
    if (e != hipSuccess) return e;
  }
  return hipSuccess;
}

}  // namespace hc
