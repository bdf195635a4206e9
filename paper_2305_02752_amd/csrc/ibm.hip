// Immersed-boundary coupling (Sec. 2.3): spreading of vertex forces onto the
// lattice and interpolation of the lattice velocity back to the vertices,
// followed by explicit Euler advection (Sec. 2.6).
//
// Kernel: Peskin's 4-point function on nodes floor(X)-1 .. floor(X)+2 per
// axis (or the 2-point linear hat on floor(X), floor(X)+1); the 3-D weight
// is the product of the per-axis weights.  Periodic axes wrap; nodes past a
// wall receive no force and read the wall velocity.
//
// Spreading and interpolation are organised by tile: one work-group per 8^3
// tile walks the list of vertices whose stencil reaches the tile (built by
// the binning kernels).  Spreading accumulates in LDS in fixed point: int32 at
// a scale of the tile, or int64 at 2^-40 with sheared images and in the reverse
// sweep; interpolation writes one partial sum per (vertex, tile) that a
// per-vertex pass adds up in a fixed order.
// Integer addition is associative, so the result is bitwise independent of
// the order in which waves and lanes arrive -- no global atomics, no
// run-to-run drift.
#include <algorithm>
#include <type_traits>

#include "ibm_dev.h"
#include "lbm_dev.h"

namespace hc {
namespace {

// Per-axis stencil of one vertex relative to a tile starting at t0: local
// node index inside the tile (-1 outside the tile or beyond a wall) and
// weight; the first node is floor(X) - 1 (K = 4) or floor(X) (K = 2).
template <int K>
__device__ inline void axis_stencil(int origin, float x, int n, int wall, int t0, int (&l)[K],
                                    float (&w)[K]) {
  const float fl = floorf(x);
  const int base = origin + (int)fl - (K == 4 ? 1 : 0);
  const float f = x - fl;
#pragma unroll
  for (int k = 0; k < K; ++k) {
    int p = base + k;
    bool in = true;
    if (wall) in = p >= 0 && p < n; else p = wrap(p, n);
    l[k] = (in && p >= t0 && p < t0 + kTile) ? p - t0 : -1;
    w[k] = stencil_w<K>(f, k);
  }
}

// Sheared periodic images (Lees-Edwards, z gradient / x flow): the image
// index of each z stencil position (floor of its unwrapped index / nz), and
// the x stencils of the vertex as seen from the first and last of them
// (x - m Delta).  Consecutive positions cross at most one boundary, so two
// x stencils cover all K.
template <int K>
struct LeStencil {
  int m[K];
  int ma, mb;
  int lxa[K], lxb[K];
  float wxa[K], wxb[K];
};

template <int K>
__device__ inline void le_stencil(const Lattice& L, int ox, float x, int oz, float zoff, int t0,
                                  LeStencil<K>& S);

// Rotate a K-entry stencil by r so that lanes holding nearby vertices visit
// different nodes at the same time (fewer LDS same-address conflicts).
template <int K>
__device__ inline void rotate(int (&l)[K], float (&w)[K], int r) {
  int l2[K];
  float w2[K];
#pragma unroll
  for (int k = 0; k < K; ++k) {
    const int src = (k + r) & (K - 1);
    l2[k] = l[0];
    w2[k] = w[0];
#pragma unroll
    for (int q = 1; q < K; ++q) {
      if (src == q) {
        l2[k] = l[q];
        w2[k] = w[q];
      }
    }
  }
#pragma unroll
  for (int k = 0; k < K; ++k) {
    l[k] = l2[k];
    w[k] = w2[k];
  }
}

template <int K>
__device__ inline void le_stencil(const Lattice& L, int ox, float x, int oz, float zoff, int t0,
                                  LeStencil<K>& S) {
  const int bz = oz + (int)floorf(zoff) - (K == 4 ? 1 : 0);
#pragma unroll
  for (int k = 0; k < K; ++k) S.m[k] = floor_div(bz + k, L.nz);
  S.ma = S.m[0];
  S.mb = S.m[K - 1];
  axis_stencil<K>(ox, x - (float)S.ma * L.le_delta, L.nx, 0, t0, S.lxa, S.wxa);
  axis_stencil<K>(ox, x - (float)S.mb * L.le_delta, L.nx, 0, t0, S.lxb, S.wxb);
}

__device__ inline void tile_origin(const Lattice& L, int t, int& x0, int& y0, int& z0) {
  x0 = (t % L.tx) * kTile;
  y0 = ((t / L.tx) % L.ty) * kTile;
  z0 = (t / (L.tx * L.ty)) * kTile;
}

// acc += trunc(q) for contributions of 2^31 or more (out of line, rare).
// Node contributions are converted to fixed point by truncation in both
// paths, so which path an entry takes never changes an integer.
__device__ __noinline__ void spread_add_wide(long long* a0, long long* a1, long long* a2, float x, float y,
                                             float z) {
  atomicAdd((unsigned long long*)a0, (unsigned long long)(long long)x);
  atomicAdd((unsigned long long*)a1, (unsigned long long)(long long)y);
  atomicAdd((unsigned long long*)a2, (unsigned long long)(long long)z);
}

// Spread phase of one tile: one thread per (vertex, tile) entry of the
// tile's list; the thread evaluates its 3 x K axis weights once and adds the
// contributions of the stencil nodes inside the tile to the LDS accumulator
// acc[3][512] (zeroed by the caller, synchronised after).
template <int K>
__device__ inline void spread_tile(const Cells& C, const Mesh& M, const Lattice& L, const Bins& B,
                                   const float* __restrict__ vec, int t, int x0, int y0, int z0,
                                   long long (*acc)[kTile * kTile * kTile]) {
  const int64_t e0 = (int64_t)t * B.cap;
  const int64_t e1 = e0 + min(B.touch_cnt[t], B.cap);
  const int rot = threadIdx.x;
  for (int64_t e = e0 + threadIdx.x; e < e1; e += blockDim.x) {
    const int v = B.touch[e] >> 5;
    const int c = v / M.nv;
    const float* o = C.off + (int64_t)v * 3;
    const float* fv = vec + (int64_t)v * 3;
    const float fx = fv[0] * kFixScaleF, fy = fv[1] * kFixScaleF, fz = fv[2] * kFixScaleF;
    int lx[K], ly[K], lz[K];
    float wx[K], wy[K], wz[K];
    LeStencil<K> S;
    le_stencil<K>(L, C.origin[3 * c + 0], o[0], C.origin[3 * c + 2], o[2], x0, S);
    rotate<K>(S.lxa, S.wxa, rot);
    rotate<K>(S.lxb, S.wxb, rot);
    axis_stencil<K>(C.origin[3 * c + 1], o[1], L.ny, L.bc[1] == 1, y0, ly, wy);
    axis_stencil<K>(C.origin[3 * c + 2], o[2], L.nz, L.bc[2] == 1, z0, lz, wz);
    rotate<K>(ly, wy, rot >> 2);
    // the x stencil of the image z position kz lies in
    auto pick_x = [&](int kz) {
      const bool a = S.m[kz] == S.ma;
#pragma unroll
      for (int kx = 0; kx < K; ++kx) {
        lx[kx] = a ? S.lxa[kx] : S.lxb[kx];
        wx[kx] = a ? S.wxa[kx] : S.wxb[kx];
      }
    };
    // weights are at most 1, so one test per entry decides whether every
    // node contribution fits the 32-bit conversion
    if (fmaxf(fabsf(fx), fmaxf(fabsf(fy), fabsf(fz))) < kFix32Max) {
#pragma unroll
      for (int kz = 0; kz < K; ++kz) {
        if (lz[kz] < 0) continue;
        pick_x(kz);
        float gx[K], gy[K], gz[K];
#pragma unroll
        for (int kx = 0; kx < K; ++kx) {
          gx[kx] = wx[kx] * fx;
          gy[kx] = wx[kx] * fy;
          gz[kx] = wx[kx] * fz;
        }
#pragma unroll
        for (int ky = 0; ky < K; ++ky) {
          if (ly[ky] < 0) continue;
          const float wzy = wz[kz] * wy[ky];
          const int row = (lz[kz] * kTile + ly[ky]) * kTile;
#pragma unroll
          for (int kx = 0; kx < K; ++kx) {
            if (lx[kx] < 0) continue;
            const int li = row + lx[kx];
            atomicAdd((unsigned long long*)&acc[0][li], (unsigned long long)(long long)(int)(wzy * gx[kx]));
            atomicAdd((unsigned long long*)&acc[1][li], (unsigned long long)(long long)(int)(wzy * gy[kx]));
            atomicAdd((unsigned long long*)&acc[2][li], (unsigned long long)(long long)(int)(wzy * gz[kx]));
          }
        }
      }
    } else {
      for (int kz = 0; kz < K; ++kz) {
        if (lz[kz] < 0) continue;
        pick_x(kz);
        for (int ky = 0; ky < K; ++ky) {
          if (ly[ky] < 0) continue;
          const float wzy = wz[kz] * wy[ky];
          const int row = (lz[kz] * kTile + ly[ky]) * kTile;
          for (int kx = 0; kx < K; ++kx) {
            if (lx[kx] < 0) continue;
            const int li = row + lx[kx];
            // the same products as the 32-bit path: wzy * (wx * f)
            spread_add_wide(&acc[0][li], &acc[1][li], &acc[2][li], wzy * (wx[kx] * fx), wzy * (wx[kx] * fy),
                            wzy * (wx[kx] * fz));
          }
        }
      }
    }
  }
}

// Interpolation phase of one tile: one thread per (vertex, tile) entry sums
// w * u over its stencil nodes inside the tile (velocities staged in su) and
// stores the partial sum in the vertex's slot.  Partials are slot-major,
// [max_touch][cells x V]: entries of neighbouring vertices with the same
// slot, which one tile mostly holds together, share cache lines.
template <int K>
__device__ inline void interp_tile(const Cells& C, const Mesh& M, const Lattice& L, const Bins& B,
                                   const float4* su, int t, int x0, int y0, int z0,
                                   float4* __restrict__ partial) {
  const int cnt = min(B.touch_cnt[t], B.cap);
  const int64_t e0 = (int64_t)t * B.cap, e1 = e0 + cnt;
  for (int64_t e = e0 + threadIdx.x; e < e1; e += blockDim.x) {
    const int code = B.touch[e];
    const int v = code >> 5, j = code & 31;
    const int c = v / M.nv;
    const float* o = C.off + (int64_t)v * 3;
    int lx[K], ly[K], lz[K];
    float wx[K], wy[K], wz[K];
    LeStencil<K> S;
    le_stencil<K>(L, C.origin[3 * c + 0], o[0], C.origin[3 * c + 2], o[2], x0, S);
    axis_stencil<K>(C.origin[3 * c + 1], o[1], L.ny, L.bc[1] == 1, y0, ly, wy);
    axis_stencil<K>(C.origin[3 * c + 2], o[2], L.nz, L.bc[2] == 1, z0, lz, wz);
    float ux = 0.f, uy = 0.f, uz = 0.f;
#pragma unroll
    for (int kz = 0; kz < K; ++kz) {
      if (lz[kz] < 0) continue;
      const bool a = S.m[kz] == S.ma;
#pragma unroll
      for (int kx = 0; kx < K; ++kx) {
        lx[kx] = a ? S.lxa[kx] : S.lxb[kx];
        wx[kx] = a ? S.wxa[kx] : S.wxb[kx];
      }
      const float shift = (float)S.m[kz] * L.le_u;   // velocity of the image this z position lies in
#pragma unroll
      for (int ky = 0; ky < K; ++ky) {
        if (ly[ky] < 0) continue;
        const float wzy = wz[kz] * wy[ky];
        const int row = (lz[kz] * kTile + ly[ky]) * kTile;
#pragma unroll
        for (int kx = 0; kx < K; ++kx) {
          if (lx[kx] < 0) continue;
          const float w = wzy * wx[kx];
          const float4 q = su[row + lx[kx]];
          ux += w * (q.x + shift);
          uy += w * q.y;
          uz += w * q.z;
        }
      }
    }
    partial[(int64_t)j * C.n * M.nv + v] = make_float4(ux, uy, uz, 0.f);
  }
}

// Which tile block b works on.  Work-groups go to the 8 XCDs round-robin by
// block id; each XCD gets one contiguous range of tiles, walked in order, so
// the neighbours a tile pulls boundary populations from were mostly just
// processed on the same XCD and sit in its L2.  -1 for padding blocks.
__device__ inline int tile_of_block(const Lattice& L, int b) {
  const int per = (L.ntiles + 7) >> 3;
  const int t = (b & 7) * per + (b >> 3);
  return t < L.ntiles ? t : -1;
}

__host__ __device__ inline int tile_grid(const Lattice& L) { return ((L.ntiles + 7) >> 3) * 8; }

// ---------------------------------------------------------------------------
// Sorted-entry form of the two immersed-boundary phases.
//
// The (vertex, tile) entries of a tile are staged in LDS as compact records:
// per axis the run of stencil positions that fall inside the tile; the
// fractional position; the vertex force.  The records are ordered by the shape of
// their in-tile box (nodes per axis), so the lanes of a wave share their
// loop bounds, and each lane walks only its entry's in-tile nodes with
// statically indexed registers.  All four stencil weights of an axis come
// from one square root: with s = sqrt(1 + 4f(1 - f)), the weights of the
// nodes floor(X) - 1 .. floor(X) + 2 are (3 - 2f - s)/8, (3 - 2f + s)/8,
// (1 + 2f + s)/8 and (1 + 2f - s)/8 (Peskin's 4-point function at
// distances 1 + f, f, 1 - f, 2 - f).
//
// Spreading accumulates in LDS as int32 fixed point (node contributions
// truncated) at a power-of-two scale chosen per tile from a bound
// on every node sum: the sum over the tile's entries of their largest force
// component times the largest weight one entry puts on one node.  The bound
// is summed in integers (each term rounded up on a 2^-bexp grid of the tile's
// largest component), so it does not depend on the order of the entries;
// integer node sums do not either, so the result is bitwise reproducible
// although the order of the records is not.
//
// With sheared images (two or more tiles along z) the nodes of one entry
// all lie in one image, so an entry is staged at its x as seen from that
// image and walks its nodes like any other; the image index is kept for the
// image's velocity.  Its forces accumulate as 2^-40 fixed-point int64, as
// do the reverse sweep's cotangents.
namespace srt {

// Records staged at once.  With 32 bytes each the work-group's LDS allows six
// per CU; 768 records (five per CU) took 2.40 ms for 2.24 on 256 x 256 x 512
// sites with 18,600 cells (475 entries per tile), 400 (eight) 2.26.
constexpr int kThreads = 256;
constexpr int kStage = 512;
constexpr int kPerThread = kStage / kThreads;
constexpr int kKeys = 64;     // box shapes: 1..4 in-tile nodes on each axis
// LDS pitch of the node arrays.  Clipped boxes start at few distinct nodes, so
// with rows of 8 and planes of 64 the lanes of a wave pile up on few banks (8.3
// cycles per LDS access, counted): counting lanes per bank over the entries of
// a dense suspension, 7.2 to 8.0 per atomic and 3.5 to 3.9 per read with
// pitches 8 and 64, 5.1 and 2.3 with 9 and 77.
constexpr int kRow = 9, kPlane = 77, kNodes = 8 * kPlane;
__device__ __forceinline__ int node_at(int i) { return (i >> 6) * kPlane + ((i >> 3) & 7) * kRow + (i & 7); }

template <bool I64>
struct Smem {
  // spread accumulator: int32 at the tile's scale, or 2^-40 int64
  typename std::conditional<I64, long long, int>::type acc[3][kNodes];
  float4 pos[kStage];       // fractions x, y, z; axis runs (bits)
  float4 force[kStage];     // force x, y, z; entry code (vertex * 32 + slot, bits)
  int cnt[kKeys];           // records per box shape, then the first record of each shape
  unsigned fmax;            // largest force component magnitude (float bits)
  int fsum;                 // sum of the entries' largest components, in units of fmax 2^-bexp
  int bad;                  // some node's velocity is not finite (4-point kernel)
  int image[I64 ? kStage : 1];   // image index of the record's nodes
  // The velocity takes the accumulator's place, each node's in the slots of
  // its own sums, so the thread that owns a node needs no other's data.
  __device__ __forceinline__ void put_u(int i, float x, float y, float z) {
    if (I64) {
      reinterpret_cast<float2*>(acc[0])[i] = make_float2(x, y);
      reinterpret_cast<float2*>(acc[1])[i].x = z;
    } else {
      reinterpret_cast<float*>(acc[0])[i] = x;
      reinterpret_cast<float*>(acc[1])[i] = y;
      reinterpret_cast<float*>(acc[2])[i] = z;
    }
  }
  __device__ __forceinline__ float3 get_u(int i) const {
    if (I64) {
      const float2 a = reinterpret_cast<const float2*>(acc[0])[i];
      return make_float3(a.x, a.y, reinterpret_cast<const float2*>(acc[1])[i].x);
    }
    return make_float3(reinterpret_cast<const float*>(acc[0])[i], reinterpret_cast<const float*>(acc[1])[i],
                       reinterpret_cast<const float*>(acc[2])[i]);
  }
};

// (16 bytes a store: 2.24 -> 2.23 ms on 256 x 256 x 512 sites, 18,600 cells)
template <bool I64>
__device__ __forceinline__ void clear_sums(Smem<I64>& S) {
  static_assert(sizeof(S.acc) % sizeof(int4) == 0, "sums in whole 16-byte words");
  for (int i = threadIdx.x; i < (int)(sizeof(S.acc) / sizeof(int4)); i += kThreads)
    reinterpret_cast<int4*>(S.acc)[i] = make_int4(0, 0, 0, 0);
}

// In-tile run along one axis: the K positions base + k (wrapped on a periodic
// axis, dropped past a wall) meet the tile's nodes [t0, t0 + 8) in one run of
// consecutive stencil indices and nodes.  Only on a periodic axis of up to
// kSmall nodes can the first tile hold nodes on both sides of the seam; the
// run is then all K positions from p0 on, see node().  Bits 0..2: first node
// - t0, 3..4: its stencil index, 5..7: count.
constexpr int kSmall = 10;
template <int K>
__device__ __forceinline__ unsigned axis_run(int base, int n, int wall, int t0) {
  int p0 = wall ? base : wrap(base, n);
  if (!wall && p0 + K > n && t0 == 0) {
    if (p0 < kTile) return (unsigned)(p0 | (K << 5));
    p0 -= n;
  }
  const int lo = max(max(p0, t0), 0), hi = min(min(p0 + K, t0 + kTile), n);
  const int c = max(hi - lo, 0);
  return c ? (unsigned)((lo - t0) | ((lo - p0) << 3) | (c << 5)) : 0u;
}

// The four weights of a fraction f from one hardware root.  Against 64 bits
// over [0, 1): at most 4.5e-8, 0.8e-8 to 1.4e-8 rms; phi4's correctly rounded
// root of a radicand with cancellation, once per weight: 7.0e-8, 1.5e-8 to
// 1.9e-8 rms.
template <int K>
__device__ __forceinline__ void weights(float f, float (&W)[4]) {
  if (K == 4) {
    const float s = __builtin_amdgcn_sqrtf(fmaf(4.f * f, 1.f - f, 1.f));
    const float a = 3.f - 2.f * f, b = 1.f + 2.f * f;
    W[0] = 0.125f * (a - s);
    W[1] = 0.125f * (a + s);
    W[2] = 0.125f * (b + s);
    W[3] = 0.125f * (b - s);
  } else {
    W[0] = 1.f - f;
    W[1] = f;
    W[2] = 0.f;
    W[3] = 0.f;
  }
}

struct Axis {
  int n, l0;
  float w[4];
};

// Run and weights of an axis of n nodes: w[s] is the weight of the run's s-th
// node.  SMALL (some axis of the lattice has up to kSmall nodes): a run across
// the seam wraps, and its nodes in the second tile weigh nothing here.
template <int K, bool SMALL>
__device__ __forceinline__ void decode(unsigned run, float f, int n, Axis& A) {
  float W[4];
  weights<K>(f, W);
  A.l0 = (int)(run & 7u);
  A.n = (int)((run >> 5) & 7u);
  const bool k1 = run & 8u, k2 = run & 16u;   // shift by the first stencil index
  const float a = k1 ? W[1] : W[0], b = k1 ? W[2] : W[1], c = k1 ? W[3] : W[2], d = W[3];
  A.w[0] = k2 ? c : a;
  A.w[1] = k2 ? d : b;
  A.w[2] = c;
  A.w[3] = d;
  if (SMALL) {
#pragma unroll
    for (int s = 0; s < 4; ++s)
      if (A.l0 + s >= kTile && A.l0 + s < n) A.w[s] = 0.f;
  }
}

// Tile-local node s of a run on an axis of n nodes.
template <bool SMALL>
__device__ __forceinline__ int node(int l0, int s, int n) {
  const int l = l0 + s;
  return SMALL ? min(l >= n ? l - n : l, kTile - 1) : l;
}

// Largest weight one entry can put on one node: the product over the axes
// of the largest per-axis weight, 1/2 for the 4-point function and 1 for
// the hat (lattice sides of at least 4 keep the K positions of an axis on
// distinct nodes).
__device__ __forceinline__ float max_node_weight(const Lattice& L) { return L.kernel == 4 ? 0.125f : 1.f; }

// Units of fmax 2^-bexp that bound an entry's largest force component fm
// from above (fm <= fmax, rfmax a reciprocal of fmax within a few ulp: the
// product is within 0.2 units, so truncating and adding one unit bounds it);
// the grid is set by the list capacity (cap 2^bexp <= 2^30), so a full
// tile list's units sum to below 2^31.
__device__ __forceinline__ int bound_units(float fm, float fmax, float rfmax, int bexp) {
  return fmax > 0.f ? (int)(fm * rfmax * ldexpf(1.f, bexp)) + 1 : 1;
}

// Exponent k of the fixed-point scale 2^k: with the entries' largest force
// components summing to at most fsum units of fmax 2^-bexp, every node sum
// stays below 2^30 (half the int32 range, which also covers the rounding of
// the weights and of the contributions).
__device__ __forceinline__ int fix_exponent(int fsum, float fmax, float wmax, int bexp) {
  const float x = (float)fsum * ldexpf(fmax, -bexp) * wmax;
  if (!(x > 0.f)) return 30;     // no force (or NaN): any scale
  if (!(x < 3.0e38f)) return 0;  // infinite force: the move's non-finite check reports it
  int e;
  frexpf(x, &e);                 // x = m 2^e, m in [0.5, 1)
  return min(max(30 - e, -100), 100);
}

// Wave-wide max / sum with DPP lane swaps inside each row of 16 lanes (xor
// 1, xor 2, then the mirrored half-row and row), and the four row results
// combined in scalar registers; every lane of the wave must be active.
template <int CTRL>
__device__ __forceinline__ int dpp_swap(int v) {
  return __builtin_amdgcn_update_dpp(0, v, CTRL, 0xF, 0xF, false);
}

__device__ __forceinline__ float wave_max(float v) {
  unsigned u = __float_as_uint(v);   // non-negative floats order as their bits
  u = max(u, (unsigned)dpp_swap<0xB1>((int)u));    // quad_perm [1,0,3,2]
  u = max(u, (unsigned)dpp_swap<0x4E>((int)u));    // quad_perm [2,3,0,1]
  u = max(u, (unsigned)dpp_swap<0x141>((int)u));   // row_half_mirror
  u = max(u, (unsigned)dpp_swap<0x140>((int)u));   // row_mirror
  const unsigned a = (unsigned)__builtin_amdgcn_readlane((int)u, 0), b = (unsigned)__builtin_amdgcn_readlane((int)u, 16);
  const unsigned c = (unsigned)__builtin_amdgcn_readlane((int)u, 32), d = (unsigned)__builtin_amdgcn_readlane((int)u, 48);
  return __uint_as_float(max(max(a, b), max(c, d)));
}

__device__ __forceinline__ int wave_sum(int v) {
  v += dpp_swap<0xB1>(v);
  v += dpp_swap<0x4E>(v);
  v += dpp_swap<0x141>(v);
  v += dpp_swap<0x140>(v);
  return __builtin_amdgcn_readlane(v, 0) + __builtin_amdgcn_readlane(v, 16) +
         __builtin_amdgcn_readlane(v, 32) + __builtin_amdgcn_readlane(v, 48);
}

__device__ __forceinline__ float entry_fmax(const Cells& C, const Bins& B, int t, int i) {
  const int v = B.touch[(int64_t)t * B.cap + i] >> 5;
  const float* fv = C.force + (int64_t)v * 3;
  return fmaxf(fabsf(fv[0]), fmaxf(fabsf(fv[1]), fabsf(fv[2])));
}

// Largest force component over entries [0, ne) of tile t into S.fmax, then
// the bound sum into S.fsum (both zeroed and synchronised by the caller).
// Each entry's largest component is gathered once and kept in the record
// space (free until the staging) when the list fits it, else gathered
// again for the sum.  Ends synchronised.
constexpr int kBoundKeep = (int)(sizeof(float4) * kStage / sizeof(float));
__device__ __forceinline__ void force_bound(const Cells& C, const Bins& B, int t, int ne, Smem<false>& S) {
  float* kept = reinterpret_cast<float*>(S.pos);
  const bool keep = ne <= kBoundKeep;
  float m = 0.f;
  for (int i = threadIdx.x; i < ne; i += blockDim.x) {
    const float f = entry_fmax(C, B, t, i);
    if (keep) kept[i] = f;
    m = fmaxf(m, f);
  }
  m = wave_max(m);
  if ((threadIdx.x & (kWave - 1)) == 0) atomicMax(&S.fmax, __float_as_uint(m));
  lds_barrier();
  const float fmx = __uint_as_float(S.fmax), rf = __builtin_amdgcn_rcpf(fmx);
  int u = 0;
  for (int i = threadIdx.x; i < ne; i += blockDim.x)
    u += bound_units(keep ? kept[i] : entry_fmax(C, B, t, i), fmx, rf, B.bexp);
  u = wave_sum(u);
  if ((threadIdx.x & (kWave - 1)) == 0) atomicAdd(&S.fsum, u);
  lds_barrier();
}

// Place of a box shape (nodes per axis less one) in the order of the
// records: z by z, alternately up and down in y and x, so that neighbouring
// shapes differ by one node on one axis.  A wave holds records of about ten
// shapes and loops to the largest count of each axis: 10% fewer nodes than
// counting up on every axis.
__device__ __forceinline__ int shape_key(int x, int y, int z) {
  y ^= z & 1 ? 3 : 0;
  const int r = z * 4 + y;
  return r * 4 + (x ^ (r & 1 ? 3 : 0));
}

// Chunks of a list longer than kStage: a first one of 1..kStage entries,
// then full ones, so that the last chunk staged for the spread is a full
// one, and it is still staged when the interpolation starts.
__device__ __forceinline__ int first_chunk(int ne) { return ne - (ne - 1) / kStage * kStage; }

// Stage entries [e0, e0 + m) of tile t (m <= kStage) as
// records ordered by box shape; with_force also stages the forces, and with
// bound as well the force bound of these entries (S.fmax, S.fsum: the whole
// tile's when they are all staged at once).  Ends synchronised.
template <int K, bool LE, bool I64>
__device__ __forceinline__ void stage(const Cells& C, const Mesh& M, const Lattice& L, const Bins& B,
                                      const float* __restrict__ vec, int t,
                             int x0, int y0, int z0, int e0, int m, bool with_force, bool bound,
                             Smem<I64>& S) {
  for (int i = threadIdx.x; i < kKeys; i += blockDim.x) S.cnt[i] = 0;
  lds_barrier();
  constexpr int R = kPerThread;
  float4 pos[R], force[R];
  int key[R], rank[R], image[R];
  float fmax = 0.f, fm[R];
  const int b = K == 4 ? -1 : 0;
  const float rnv = __builtin_amdgcn_rcpf((float)M.nv);
#pragma unroll
  for (int h = 0; h < R; ++h) {
    const int i = (int)threadIdx.x + h * kThreads;
    key[h] = -1;
    rank[h] = 0;
    image[h] = 0;
    fm[h] = 0.f;
    pos[h] = make_float4(0.f, 0.f, 0.f, 0.f);
    force[h] = make_float4(0.f, 0.f, 0.f, 0.f);
    if (i < m) {
      const int code = B.touch[(int64_t)t * B.cap + e0 + i];
      const int v = code >> 5, c = div_small(v, M.nv, rnv);
      const float* o = C.off + (int64_t)v * 3;
      float ox = o[0];
      const float oy = o[1], oz = o[2];
      const float fy = floorf(oy), fz = floorf(oz);
      const int bz = C.origin[3 * c + 2] + (int)fz + b;
      const unsigned rz = axis_run<K>(bz, L.nz, L.bc[2] == 1, z0);
      if (LE) {   // the image of the first in-tile z node is that of all of them
        image[h] = floor_div(bz + (int)((rz >> 3) & 3u), L.nz);
        ox = fmaf(-(float)image[h], L.le_delta, ox);
      }
      const float fx = floorf(ox);
      const unsigned rx = axis_run<K>(C.origin[3 * c] + (int)fx + b, L.nx, L.bc[0] == 1, x0);
      const unsigned ry = axis_run<K>(C.origin[3 * c + 1] + (int)fy + b, L.ny, L.bc[1] == 1, y0);
      pos[h] = make_float4(ox - fx, oy - fy, oz - fz, __uint_as_float(rx | (ry << 8) | (rz << 16)));
      force[h].w = __int_as_float(code);
      if (with_force) {
        const float* fv = vec + (int64_t)v * 3;
        force[h].x = fv[0];
        force[h].y = fv[1];
        force[h].z = fv[2];
        fm[h] = fmaxf(fabsf(fv[0]), fmaxf(fabsf(fv[1]), fabsf(fv[2])));
        fmax = fmaxf(fmax, fm[h]);
      }
      key[h] = shape_key(max((int)(rx >> 5), 1) - 1, max((int)(ry >> 5), 1) - 1, max((int)(rz >> 5), 1) - 1);
      rank[h] = atomicAdd(&S.cnt[key[h]], 1);
    }
  }
  if (bound) {
    const float w = wave_max(fmax);
    if ((threadIdx.x & (kWave - 1)) == 0) atomicMax(&S.fmax, __float_as_uint(w));
  }
  lds_barrier();
  if (bound) {   // S.fmax is complete: the bound sum (read after the final barrier)
    const float fmx = __uint_as_float(S.fmax), rf = __builtin_amdgcn_rcpf(fmx);
    int u = 0;
#pragma unroll
    for (int h = 0; h < R; ++h)
      if (key[h] >= 0) u += bound_units(fm[h], fmx, rf, B.bexp);
    u = wave_sum(u);
    if ((threadIdx.x & (kWave - 1)) == 0) atomicAdd(&S.fsum, u);
  }
  if (threadIdx.x < kKeys) {   // first record of each shape: exclusive scan in the first wave
    const int own = S.cnt[threadIdx.x];
    int v = own;
#pragma unroll
    for (int d = 1; d < kKeys; d <<= 1) {
      const int u = __shfl_up(v, d);
      if ((int)threadIdx.x >= d) v += u;
    }
    S.cnt[threadIdx.x] = v - own;
  }
  lds_barrier();
#pragma unroll
  for (int h = 0; h < R; ++h) {
    if (key[h] < 0) continue;
    const int p = S.cnt[key[h]] + rank[h];
    S.pos[p] = pos[h];
    S.force[p] = force[h];
    if (LE) S.image[p] = image[h];
  }
  lds_barrier();
}

// Spread the m staged records into S.acc at the scale 2^kexp.  Node
// contributions are truncated (RN false) or rounded to nearest (RN true).
// A node sum's error is then at most one unit per contribution, or about
// the square root of the contributions times half a unit; the unit grows
// with the tile's force bound, i.e. with its entries, so crowded tiles
// (more than kRoundAbove entries) round.
// The int64 sums truncate at 2^40 (scale): forces of 2^-9
// and more take the full-range conversion (WIDE), a truncation as well, so
// which of the two an entry takes never changes an integer.
constexpr int kRoundAbove = 1024;
template <int K, bool RN, bool WIDE, bool SMALL, bool I64>
__device__ __forceinline__ void spread_entries(int m, const Lattice& L, float scale, Smem<I64>& S) {
  auto add = [&](int comp, int li, float q) {
    if (I64) {
      const long long n = WIDE ? (long long)q : (long long)(int)q;
      atomicAdd(reinterpret_cast<unsigned long long*>(&S.acc[comp][li]), (unsigned long long)n);
    } else {
      atomicAdd(reinterpret_cast<int*>(&S.acc[comp][li]), RN ? __float2int_rn(q) : (int)q);
    }
  };
  for (int i = threadIdx.x; i < m; i += blockDim.x) {
    const float4 pos = S.pos[i], force = S.force[i];
    const unsigned run = __float_as_uint(pos.w);
    Axis X, Y, Z;
    decode<K, SMALL>(run, pos.x, L.nx, X);
    decode<K, SMALL>(run >> 8, pos.y, L.ny, Y);
    decode<K, SMALL>(run >> 16, pos.z, L.nz, Z);
    const float fx = force.x * scale, fy = force.y * scale, fz = force.z * scale;
    float gx[K], gy[K], gz[K];
#pragma unroll
    for (int s = 0; s < K; ++s) {
      gx[s] = X.w[s] * fx;
      gy[s] = X.w[s] * fy;
      gz[s] = X.w[s] * fz;
    }
#pragma unroll
    for (int iz = 0; iz < K; ++iz) {
      if (iz >= Z.n) continue;
#pragma unroll
      for (int iy = 0; iy < K; ++iy) {
        if (iy >= Y.n) continue;
        const float wzy = Z.w[iz] * Y.w[iy];
        const int row = node<SMALL>(Z.l0, iz, L.nz) * kPlane + node<SMALL>(Y.l0, iy, L.ny) * kRow;
#pragma unroll
        for (int ix = 0; ix < K; ++ix) {
          if (ix >= X.n) continue;
          const int li = row + node<SMALL>(X.l0, ix, L.nx);
          add(0, li, wzy * gx[ix]);
          add(1, li, wzy * gy[ix]);
          add(2, li, wzy * gz[ix]);
        }
      }
    }
  }
}

template <int K, bool SMALL, bool I64>
__device__ __forceinline__ void spread(int m, const Lattice& L, int ne, int kexp, Smem<I64>& S) {
  if constexpr (I64) {
    bool wide = false;   // the wave's choice: any of its forces
    for (int i = threadIdx.x; i < m; i += kThreads) {
      const float4 f = S.force[i];
      wide = wide || !(fmaxf(fabsf(f.x), fmaxf(fabsf(f.y), fabsf(f.z))) * kFixScaleF < kFix32Max);
    }
    if (__any(wide)) spread_entries<K, false, true, SMALL>(m, L, kFixScaleF, S);
    else spread_entries<K, false, false, SMALL>(m, L, kFixScaleF, S);
  } else {
    if (ne > kRoundAbove) spread_entries<K, true, false, SMALL>(m, L, ldexpf(1.f, kexp), S);
    else spread_entries<K, false, false, SMALL>(m, L, ldexpf(1.f, kexp), S);
  }
}

// Interpolation partial sums of the m staged records from the velocity
// held in S.acc (float bits), summed over the in-tile nodes in stencil
// order, into the records' partial-sum slots.
// With sheared images every node carries its image's velocity.
// CLIP: x slots past the entry's count, whose weight is zero, read its first
// node again: a node outside the stencil may not reach the vertex, and 0 x NaN
// would.  Without it they read on along the row, so that a row's reads share
// one address; that is for tiles whose velocities are all finite.  With two
// nodes a row the select costs less than the test for them (a pass of 240 tiles
// 13.94 us for 14.20).
template <int K, bool SMALL, bool CLIP, bool LE>
__device__ __forceinline__ void interp(int m, const Lattice& L, const Smem<LE>& S, int64_t stride,
                                       float4* __restrict__ partial) {
  for (int i = threadIdx.x; i < m; i += blockDim.x) {
    const float4 pos = S.pos[i];
    const unsigned run = __float_as_uint(pos.w);
    Axis X, Y, Z;
    decode<K, SMALL>(run, pos.x, L.nx, X);
    decode<K, SMALL>(run >> 8, pos.y, L.ny, Y);
    decode<K, SMALL>(run >> 16, pos.z, L.nz, Z);
    // x slots past the entry's count carry weight zero, so a row's reads have
    // no branch and issue together
    float wx[K];
#pragma unroll
    for (int s = 0; s < K; ++s) wx[s] = s < X.n ? X.w[s] : 0.f;
    const float shift = LE ? (float)S.image[i] * L.le_u : 0.f;
    float sx = 0.f, sy = 0.f, sz = 0.f;
#pragma unroll
    for (int iz = 0; iz < K; ++iz) {
      if (iz >= Z.n) continue;
#pragma unroll
      for (int iy = 0; iy < K; ++iy) {
        if (iy >= Y.n) continue;
        const float wzy = Z.w[iz] * Y.w[iy];
        const int row = node<SMALL>(Z.l0, iz, L.nz) * kPlane + node<SMALL>(Y.l0, iy, L.ny) * kRow;
        float rx = 0.f, ry = 0.f, rz = 0.f;
#pragma unroll
        for (int ix = 0; ix < K; ++ix) {
          const float3 u = S.get_u(row + node<SMALL>(X.l0, CLIP && ix >= X.n ? 0 : ix, L.nx));
          rx += wx[ix] * (LE ? u.x + shift : u.x);
          ry += wx[ix] * u.y;
          rz += wx[ix] * u.z;
        }
        sx += wzy * rx;
        sy += wzy * ry;
        sz += wzy * rz;
      }
    }
    const int code = __float_as_int(S.force[i].w);
    const int v = code >> 5, j = code & 31;
    partial[(int64_t)j * stride + v] = make_float4(sx, sy, sz, 0.f);
  }
}

}  // namespace srt

// Spreading of a vertex field alone (the reverse sweep spreads cotangents
// with it): writes body * g + the spread field, tile-major (padding slots
// receive body * g).  Its entries are staged and sorted like the lattice
// pass's, in int64 sums: one box of 32^3 14 us, 24.5 with a thread per unsorted
// entry testing every node; 64 boxes of 48^3 53 and 61.  Its weights are
// srt::weights, no further off than phi4's: p . dL/dp of 24 fits of one box
// (sides 24 to 45, 40 or 60 steps) is on average 9.4e-7 off 64 bits with either.
template <int K, class CT, class MT, class LT, class BT>
__device__ __forceinline__ void spread_body(CT C, MT M, LT L, BT B, const float* __restrict__ vec, float body,
                                            float* __restrict__ F) {
  __shared__ srt::Smem<true> S;
  const int t = blockIdx.x;
  int x0, y0, z0;
  tile_origin(L, t, x0, y0, z0);
  srt::clear_sums(S);
  const int ne = min(B.touch_cnt[t], B.cap);
  lds_barrier();
  const bool small = min(L.nx, min(L.ny, L.nz)) <= srt::kSmall;
  for (int e0 = 0; e0 < ne; e0 += srt::kStage) {
    const int m = min(ne - e0, srt::kStage);
    srt::stage<K, false>(C, M, L, B, vec, t, x0, y0, z0, e0, m, true, false, S);
    if (small) srt::spread<K, true>(m, L, ne, 0, S);
    else srt::spread<K, false>(m, L, ne, 0, S);
    lds_barrier();
  }
  // every thread has used the count: leave it zero for the next binning
  if (ne > 0 && threadIdx.x == 0) B.touch_cnt[t] = 0;

  const int64_t NP = L.np, h0 = (int64_t)t * 512;
  for (int i = threadIdx.x; i < kTile * kTile * kTile; i += blockDim.x) {
    const int li = srt::node_at(i);
    F[h0 + i] = body * L.g[0] + (float)((double)S.acc[0][li] * kFixInv);
    F[NP + h0 + i] = body * L.g[1] + (float)((double)S.acc[1][li] * kFixInv);
    F[2 * NP + h0 + i] = body * L.g[2] + (float)((double)S.acc[2][li] * kFixInv);
  }
}

template <int K>
__global__ __launch_bounds__(256) void k_spread(Cells C, Mesh M, Lattice L, Bins B,
                                                const float* __restrict__ vec, float body,
                                                float* __restrict__ F) {
  spread_body<K, Cells, Mesh, Lattice, Bins>(C, M, L, B, vec, body, F);
}

template <int K>
__global__ __launch_bounds__(256) void k_spread_multi(const SpreadArgs* __restrict__ many) {
  const SpreadArgs& a = launch_record(many, blockIdx.y);
  spread_body<K, const Cells&, const Mesh&, const Lattice&, const Bins&>(a.C, a.M, a.L, a.B, a.vec, a.body, a.F);
}

constexpr int kNoWall = -1;

// The fused lattice pass, one work-group per tile, with the sorted-entry IBM
// phases (WA: the wall axis or kNoWall; SMALL: some axis has up to srt::kSmall
// nodes; LE: with sheared images and two or more tiles along z, which leave an
// entry's nodes in one image):
//  1. stage the tile's entries (records ordered by in-tile box shape) and
//     spread their forces into LDS (int32 fixed point at the tile's scale);
//  2. pull-stream + collide the tile's nodes (force = body force + spread
//     field), store their post-collision populations and keep (u, rho) in
//     LDS (writing the force and (u, rho) fields out when fields is
//     non-zero); a site whose byte in mask (when given) is non-zero lies
//     inside a cell and relaxes at L.omega_in of its highest set bit (the
//     most viscous class containing it), and its byte is cleared;
//  3. interpolate u to the staged entries into their partial-sum slots.
// Bound by the node loops of 1 and 3 (LDS atomics and reads, then the vector
// instructions around them), not by the populations' traffic: with the padded
// pitch, the up-and-down record order, 32-byte records and barriers that wait
// for LDS only, 2.77 -> 2.24 ms on 256 x 256 x 512 sites with 18,600 cells
// (the populations alone take 0.86 at copy rate), 64 -> 55 us on a walled
// 128 x 64 x 64 with 220, 379 -> 224 us with sheared images on 128^3 with 1160.
// Tiles with more entries than the LDS stages at once take them in chunks
// (the scale then comes from a first pass over all their forces, and the
// interpolation stages again every chunk but the last).
// The struct arguments come by value from the single-box kernel (its own
// parameters) and by reference to constant memory from the batched one
// (launch_record: 60 vector registers, 106 through a plain reference; with
// six waves per SIMD then 238 us for 255 on 64 boxes of 48^3): a reference to
// a kernel's by-value parameter, or a by-value copy of a record in global
// memory, would put the lattice record in scratch.  The wall axis is a
// compile-time choice of both (the boxes of a launch share it): 52.5 us for
// 54.5 on a walled 128 x 64 x 64, 19.6 for 21.4 on 32^3, 234 for 238 on the 64
// boxes.
template <int K, int WA, bool SMALL, bool LE, class CT, class MT, class LT, class BT>
__device__ __forceinline__ void tile_step_sorted_body(CT C, MT M, LT L, BT B,
                                                      const float* __restrict__ gin,
                                                      float* __restrict__ gout, float* __restrict__ F,
                                                      float4* __restrict__ macro,
                                                      float4* __restrict__ partial, int fields,
                                                      unsigned char* __restrict__ mask) {
  __shared__ srt::Smem<LE> S;
  constexpr bool W = WA != kNoWall;
  constexpr int wa = WA;
  const int t = tile_of_block(L, blockIdx.x);
  if (t < 0) return;
  int x0, y0, z0;
  tile_origin(L, t, x0, y0, z0);
  srt::clear_sums(S);
  if (threadIdx.x == 0) {
    S.fmax = 0u;
    S.fsum = 0;
    S.bad = 0;
  }
  const int ne = C.n > 0 ? min(B.touch_cnt[t], B.cap) : 0;
  __syncthreads();
  // every thread has read the count: leave it zero for the next binning
  if (ne > 0 && threadIdx.x == 0) B.touch_cnt[t] = 0;
  int kexp = 0;
  if (ne > 0) {
    // the scale must cover every chunk (the int64 sums need none)
    const bool bound = !LE && ne <= srt::kStage;
    if constexpr (!LE)
      if (!bound) srt::force_bound(C, B, t, ne, S);
    for (int e0 = 0, m = srt::first_chunk(ne); e0 < ne; e0 += m, m = srt::kStage) {
      srt::stage<K, LE>(C, M, L, B, C.force, t, x0, y0, z0, e0, m, true, bound, S);
      if (!LE && e0 == 0)
        kexp = srt::fix_exponent(S.fsum, __uint_as_float(S.fmax), srt::max_node_weight(L), B.bexp);
      srt::spread<K, SMALL>(m, L, ne, kexp, S);
      __syncthreads();
    }
  }

  const int64_t NP = L.np, h0 = (int64_t)t * 512;
  // The tile-major site index is separable, site = Sx(x) + Sy(y) + Sz(z), so
  // the pull source x - e_q of every direction is two additions of the
  // parts of the node and its neighbours (wrapped) along each axis.  Site
  // indices stay below 2^30, so they serve as 32-bit element offsets.
  const unsigned py = (unsigned)L.tx << 9, pz = py * (unsigned)L.ty;
  for (int i = threadIdx.x; i < kTile * kTile * kTile; i += blockDim.x) {
    const int x = x0 + (i & 7), y = y0 + ((i >> 3) & 7), z = z0 + (i >> 6), li = srt::node_at(i);
    if (x >= L.nx || y >= L.ny || z >= L.nz) {
      S.put_u(li, 0.f, 0.f, 0.f);
      continue;
    }
    const int xm = x == 0 ? L.nx - 1 : x - 1, xp = x == L.nx - 1 ? 0 : x + 1;
    const int ym = y == 0 ? L.ny - 1 : y - 1, yp = y == L.ny - 1 ? 0 : y + 1;
    const int zm = z == 0 ? L.nz - 1 : z - 1, zp = z == L.nz - 1 ? 0 : z + 1;
    // parts of the source coordinate x - e for e = -1, 0, +1
    const unsigned SX[3] = {(unsigned)(((xp >> 3) << 9) | (xp & 7)), (unsigned)(((x >> 3) << 9) | (x & 7)),
                            (unsigned)(((xm >> 3) << 9) | (xm & 7))};
    const unsigned SY[3] = {(unsigned)(yp >> 3) * py + (unsigned)((yp & 7) << 3),
                            (unsigned)(y >> 3) * py + (unsigned)((y & 7) << 3),
                            (unsigned)(ym >> 3) * py + (unsigned)((ym & 7) << 3)};
    const unsigned SZ[3] = {(unsigned)(zp >> 3) * pz + (unsigned)((zp & 7) << 6),
                            (unsigned)(z >> 3) * pz + (unsigned)((z & 7) << 6),
                            (unsigned)(zm >> 3) * pz + (unsigned)((zm & 7) << 6)};
    const unsigned hl = SX[1] + SY[1] + SZ[1];   // this node's site
    // wall layers: a source past the wall is the opposite population at the node itself
    bool lo = false, hi = false;
    if (W) {
      const int c = wa == 0 ? x : (wa == 1 ? y : z);
      const int n = wa == 0 ? L.nx : (wa == 1 ? L.ny : L.nz);
      lo = c == 0;
      hi = c == n - 1;
    }
    float g[kQ];
#pragma unroll
    for (int q = 0; q < kQ; ++q) {
      const unsigned src = SX[lbm::cx[q] + 1] + SY[lbm::cy[q] + 1] + SZ[lbm::cz[q] + 1];
      if (W) {
        const int ew = wa == 0 ? lbm::cx[q] : (wa == 1 ? lbm::cy[q] : lbm::cz[q]);
        const bool past = (ew == 1 && lo) || (ew == -1 && hi);
        g[q] = past ? gin[(int64_t)lbm::opp[q] * NP + hl] : gin[(int64_t)q * NP + src];
      } else if (LE && !L.le_raw && ((lbm::cz[q] > 0 && z == 0) || (lbm::cz[q] < 0 && z == L.nz - 1))) {
        g[q] = lbm::le_pull(L, gin, q, x, y);   // across the sheared boundary: whole waves
      } else {
        g[q] = (gin + (int64_t)q * NP)[src];
      }
    }
    // each thread reads and then overwrites only its own nodes' slots
    auto sum = [&](int d) {
      return LE ? (float)((double)S.acc[d][li] * kFixInv) : ldexpf((float)S.acc[d][li], -kexp);
    };
    const float fx = L.g[0] + sum(0), fy = L.g[1] + sum(1), fz = L.g[2] + sum(2);
    float rho, ux, uy, uz;
    const int64_t h = h0 + i;
    float omega = L.omega;
    if (mask) {
      const unsigned b = mask[h];
      if (b) {   // inside a cell: the most viscous class containing the site
        omega = L.omega_in[31 - __clz(b)];
        mask[h] = 0;
      }
    }
    lbm::collide(g, fx, fy, fz, omega, rho, ux, uy, uz);
    S.put_u(li, ux, uy, uz);
    if (K == 4 && !(fabsf(ux) + fabsf(uy) + fabsf(uz) < 3e38f)) S.bad = 1;
    if (fields) {
      macro[h] = make_float4(ux, uy, uz, rho);
      F[h] = fx;
      F[NP + h] = fy;
      F[2 * NP + h] = fz;
    }
#pragma unroll
    for (int q = 0; q < kQ; ++q) {
      float v = g[q];
      if (W) {   // the value heading into a moving wall carries Ladd's term
        const int ew = wa == 0 ? lbm::cx[q] : (wa == 1 ? lbm::cy[q] : lbm::cz[q]);
        if (ew == -1 && lo) v += L.wc_lo[q] * rho;
        if (ew == 1 && hi) v += L.wc_hi[q] * rho;
      }
      // streamed out past the caches: the next step reads these values
      // back only after every tile has written (measured 2.875 -> 2.823 ms)
      __builtin_nontemporal_store(v, (gout + (int64_t)q * NP) + h);
    }
  }
  if (ne == 0) return;
  lds_barrier();   // the velocities; the populations' stores need no wait
  const int64_t stride = (int64_t)C.n * M.nv;
  const bool clip = K == 2 || __builtin_amdgcn_readfirstlane(S.bad);
  auto interp = [&](int m) {
    if (clip) srt::interp<K, SMALL, true>(m, L, S, stride, partial);
    else srt::interp<K, SMALL, false>(m, L, S, stride, partial);
  };
  if (ne <= srt::kStage) {
    interp(ne);
  } else {
    // the last chunk of the spread is still staged; the others stage again
    interp(srt::kStage);
    lds_barrier();
    for (int e0 = 0, m = srt::first_chunk(ne); e0 < ne - srt::kStage; e0 += m, m = srt::kStage) {
      srt::stage<K, LE>(C, M, L, B, C.force, t, x0, y0, z0, e0, m, false, false, S);
      interp(m);
      lds_barrier();
    }
  }
}

template <int K, int WA, bool SMALL>
__global__ __launch_bounds__(256) __attribute__((amdgpu_waves_per_eu(6))) void k_tile_step_sorted(
    Cells C, Mesh M, Lattice L, Bins B,
                                                          const float* __restrict__ gin,
                                                          float* __restrict__ gout,
                                                          float* __restrict__ F,
                                                          float4* __restrict__ macro,
                                                          float4* __restrict__ partial, int fields,
                                                          unsigned char* __restrict__ mask) {
  tile_step_sorted_body<K, WA, SMALL, false, Cells, Mesh, Lattice, Bins>(C, M, L, B, gin, gout, F, macro, partial, fields,
                                                                 mask);
}

// Sheared images.  The entry-parallel form below tests every axis slot at
// every node and keeps its entries unsorted: 379 us on 128^3 with 1160 cells,
// this one 224 us.  Bound by the 64-bit LDS atomics of the spread.
template <int K, bool SMALL>
__global__ __launch_bounds__(256) void k_tile_step_sorted_le(Cells C, Mesh M, Lattice L, Bins B,
                                                             const float* __restrict__ gin,
                                                             float* __restrict__ gout, float* __restrict__ F,
                                                             float4* __restrict__ macro,
                                                             float4* __restrict__ partial, int fields,
                                                             unsigned char* __restrict__ mask) {
  tile_step_sorted_body<K, kNoWall, SMALL, true, Cells, Mesh, Lattice, Bins>(C, M, L, B, gin, gout, F, macro, partial, fields,
                                                                    mask);
}

// Batched form: box blockIdx.y.
template <int K, int WA, bool SMALL>
__global__ __launch_bounds__(256) __attribute__((amdgpu_waves_per_eu(6))) void k_tile_step_sorted_multi(const TileStepArgs* __restrict__ many) {
  const TileStepArgs& a = launch_record(many, blockIdx.y);
  tile_step_sorted_body<K, WA, SMALL, false, const Cells&, const Mesh&, const Lattice&, const Bins&>(
      a.C, a.M, a.L, a.B, a.gin, a.gout, a.F, a.macro, a.partial, a.fields, a.mask);
}

// The fused lattice pass with sheared images on a lattice of a single tile
// along z, whose entries may reach nodes of two images in the one tile: one
// thread per entry, each z node in its own image.
template <int K>
__global__ __launch_bounds__(256) void k_tile_step_le_thin(Cells C, Mesh M, Lattice L, Bins B,
                                                           const float* __restrict__ gin,
                                                           float* __restrict__ gout,
                                                           float* __restrict__ F,
                                                           float4* __restrict__ macro,
                                                           float4* __restrict__ partial, int fields,
                                                           unsigned char* __restrict__ mask) {
  __shared__ long long acc[3][kTile * kTile * kTile];
  __shared__ float4 su[kTile * kTile * kTile];
  const int t = tile_of_block(L, blockIdx.x);
  if (t < 0) return;
  int x0, y0, z0;
  tile_origin(L, t, x0, y0, z0);
  for (int i = threadIdx.x; i < kTile * kTile * kTile; i += blockDim.x) {
    acc[0][i] = 0;
    acc[1][i] = 0;
    acc[2][i] = 0;
  }
  __syncthreads();
  if (C.n > 0) spread_tile<K>(C, M, L, B, C.force, t, x0, y0, z0, acc);
  __syncthreads();

  const int64_t NP = L.np, h0 = (int64_t)t * 512;
  for (int i = threadIdx.x; i < kTile * kTile * kTile; i += blockDim.x) {
    const int x = x0 + (i & 7), y = y0 + ((i >> 3) & 7), z = z0 + (i >> 6);
    if (x >= L.nx || y >= L.ny || z >= L.nz) {
      su[i] = make_float4(0.f, 0.f, 0.f, 0.f);
      continue;
    }
    float g[kQ];
#pragma unroll
    for (int q = 0; q < kQ; ++q) {
      if (!L.le_raw && ((lbm::cz[q] > 0 && z == 0) || (lbm::cz[q] < 0 && z == L.nz - 1))) {
        g[q] = lbm::le_pull(L, gin, q, x, y);
      } else {
        int qs;
        const int64_t src = lbm::pull_source(L, q, x, y, z, &qs);
        g[q] = gin[qs * NP + src];
      }
    }
    const float fx = L.g[0] + (float)((double)acc[0][i] * kFixInv);
    const float fy = L.g[1] + (float)((double)acc[1][i] * kFixInv);
    const float fz = L.g[2] + (float)((double)acc[2][i] * kFixInv);
    float rho, ux, uy, uz;
    const int64_t h = h0 + i;
    float omega = L.omega;
    if (mask) {
      const unsigned b = mask[h];
      if (b) {   // inside a cell: the most viscous class containing the site
        omega = L.omega_in[31 - __clz(b)];
        mask[h] = 0;
      }
    }
    lbm::collide(g, fx, fy, fz, omega, rho, ux, uy, uz);
    const float4 m = make_float4(ux, uy, uz, rho);
    su[i] = m;
    if (fields) {
      macro[h] = m;
      F[h] = fx;
      F[NP + h] = fy;
      F[2 * NP + h] = fz;
    }
#pragma unroll
    for (int q = 0; q < kQ; ++q) gout[q * NP + h] = g[q] + lbm::wall_coeff(L, q, x, y, z) * rho;
  }
  if (C.n == 0) return;
  __syncthreads();
  interp_tile<K>(C, M, L, B, su, t, x0, y0, z0, partial);
  __syncthreads();   // every thread has read the count: leave it zero for the next binning
  if (threadIdx.x == 0) B.touch_cnt[t] = 0;
}

template <int K>
__global__ __launch_bounds__(256) void k_advect(Cells C, Mesh M, Lattice L, Bins B,
                                                const float4* __restrict__ partial,
                                                int* __restrict__ flags, int ab2) {
  const int64_t v = (int64_t)blockIdx.x * blockDim.x + threadIdx.x;
  if (v >= (int64_t)C.n * M.nv) return;
  float nx[3];
  ibmd::advect_vertex<K>(C, M, L, B, partial, flags, v, nx, nullptr, ab2 != 0);
}

}  // namespace

// f(whether the lattice needs the wrapping form, as a compile-time constant).
// One form per kernel: with both in one, a pass over 240 tiles of few entries
// (2-point kernel, 91 x 25 x 40, 27 cells) took 14.0 us for 13.9.
template <class F>
static void with_small(const Lattice& L, F f) {
  if (std::min(L.nx, std::min(L.ny, L.nz)) <= srt::kSmall) f(std::true_type());
  else f(std::false_type());
}

// The reverse sweep differentiates the 4-point function; the spread and the
// batched launches are part of it and have no 2-point form.
hipError_t launch_spread_vec(const Cells& c, const Mesh& m, const Lattice& L, const Bins& b,
                             const float* vec, float body, float* F, hipStream_t s) {
  if (L.kernel != 4) return hipErrorInvalidValue;
  hipLaunchKernelGGL(k_spread<4>, dim3(L.ntiles), dim3(256), 0, s, c, m, L, b, vec, body, F);
  return hipGetLastError();
}

hipError_t launch_spread_vec_multi(const SpreadArgs& a0, const SpreadArgs* dev, int n, hipStream_t s) {
  if (n == 0) return hipSuccess;
  if (a0.L.kernel != 4) return hipErrorInvalidValue;
  hipLaunchKernelGGL(k_spread_multi<4>, dim3((unsigned)a0.L.ntiles, (unsigned)n), dim3(256), 0, s, dev);
  return hipGetLastError();
}

// Boxes of one shape and one set of boundaries, without sheared images.
hipError_t launch_tile_step_multi(const TileStepArgs& a0, const TileStepArgs* dev, int n, hipStream_t s) {
  if (n == 0) return hipSuccess;
  if (a0.L.le || a0.L.kernel != 4) return hipErrorInvalidValue;
  auto go = [&](auto kern) {
    hipLaunchKernelGGL(kern, dim3((unsigned)tile_grid(a0.L), (unsigned)n), dim3(256), 0, s, dev);
  };
  with_small(a0.L, [&](auto small) {
    constexpr bool S = decltype(small)::value;
    if (a0.L.wall_axis == 0) go(k_tile_step_sorted_multi<4, 0, S>);
    else if (a0.L.wall_axis == 1) go(k_tile_step_sorted_multi<4, 1, S>);
    else if (a0.L.wall_axis == 2) go(k_tile_step_sorted_multi<4, 2, S>);
    else go(k_tile_step_sorted_multi<4, kNoWall, S>);
  });
  return hipGetLastError();
}

hipError_t launch_tile_step(const Cells& c, const Mesh& m, const Lattice& L, const Bins& b,
                            const float* gin, float* gout, float* F, float4* macro, float4* partial,
                            bool fields, unsigned char* mask, hipStream_t s) {
  auto go = [&](auto kern) {
    hipLaunchKernelGGL(kern, dim3((unsigned)tile_grid(L)), dim3(256), 0, s, c, m, L, b, gin, gout, F, macro, partial,
                       fields ? 1 : 0, mask);
  };
  auto form = [&](auto k, auto small) {
    constexpr int K = decltype(k)::value;
    constexpr bool S = decltype(small)::value;
    if (L.le && L.tz == 1) go(k_tile_step_le_thin<K>);   // an entry's nodes may lie in two images
    else if (L.le) go(k_tile_step_sorted_le<K, S>);
    else if (L.wall_axis == 0) go(k_tile_step_sorted<K, 0, S>);
    else if (L.wall_axis == 1) go(k_tile_step_sorted<K, 1, S>);
    else if (L.wall_axis == 2) go(k_tile_step_sorted<K, 2, S>);
    else go(k_tile_step_sorted<K, kNoWall, S>);
  };
  with_small(L, [&](auto small) {
    if (L.kernel == 4) form(std::integral_constant<int, 4>(), small);
    else form(std::integral_constant<int, 2>(), small);
  });
  return hipGetLastError();
}

hipError_t launch_advect(const Cells& c, const Mesh& m, const Lattice& L, const Bins& b,
                         const float4* partial, int* flags, bool ab2, hipStream_t s) {
  const int64_t n = (int64_t)c.n * m.nv;
  if (n == 0) return hipSuccess;
  const dim3 gv((unsigned)((n + 255) / 256));
  const int a2 = ab2 ? 1 : 0;
  if (L.kernel == 4)
    hipLaunchKernelGGL(k_advect<4>, gv, dim3(256), 0, s, c, m, L, b, partial, flags, a2);
  else
    hipLaunchKernelGGL(k_advect<2>, gv, dim3(256), 0, s, c, m, L, b, partial, flags, a2);
  return hipGetLastError();
}

}  // namespace hc
