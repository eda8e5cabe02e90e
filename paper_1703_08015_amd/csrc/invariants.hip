// Projection of a starting state onto the invariants of a start from rest.
//
// Mass: rho is rescaled per lattice-connected component so that it holds
// rho0 per node.  Staggered momentum: the invariants are the functionals
// sum_x beta(x).j(x) with beta in the null space of the link operator
// (A beta)_link = c.beta(x+c) + c.beta(x); the operator
//   (T j)(x) = 3 sum_{i: x + c_i fluid} w_i c_i [c_i.(j(x) + j(x + c_i))] / 2
// equals (3/2) A^T W A, so its range is orthogonal to all of them, and the
// Richardson sweeps j <- j + T(rho u - j) from j = 0 give a momentum field
// with none of them while approaching rho u (T is the identity on smooth
// fields in the bulk, with eigenvalues in [0, 1]).
//
// The sweeps carry the residual r = rho u - j, for which a sweep is
// r <- r - T r: one field of three components to read at the 18 neighbours
// instead of rho, u and j, and u = (rho u - r) / rho at the end.
//
// Launches on the caller's stream: clear the per-component sums, sum
// (rho, 1) per component, rescale rho, one stencil launch per sweep
// (ping-pong buffers in the scratch), the last of which writes u.
// Per-component sums: a wavefront keeps two components in registers over a stride
// of nodes, and a workgroup adds one total (112 x 104 x 96 at porosity 0.5: 420 ->
// 11 us against one FP64 atomic pair per 64 nodes, all on one address; 128^3 with
// 14,524 pockets in 5% of the nodes: 24 -> 20 us, with 10,080 components in 12%:
// 700 -> 106 us).
#include <hip/hip_runtime.h>

#include <algorithm>
#include <mutex>

#include "device.h"
#include "internal.h"

using lbm::set_error;

namespace {

constexpr int kBlock = 256;
constexpr int kMaxIterations = 1000;

// Labels outside [0, count) are treated as solid: a bad label array leaves
// its nodes untouched instead of adding out of bounds.
__device__ inline int checked(int32_t label, int32_t count) { return label < count ? label : -1; }

__global__ void __launch_bounds__(kBlock) k_clear(double *p, int64_t n) {
  for (int64_t i = blockIdx.x * (int64_t)kBlock + threadIdx.x; i < n; i += (int64_t)gridDim.x * kBlock) p[i] = 0.0;
}

// (rho, 1) summed per component.  A wavefront goes over its nodes 64 at a time and
// holds the sums of two components, per lane, in registers: a, the one that it
// has met again and again, and b, the largest other one of the last 64 nodes
// that had neither (which becomes a when it comes again where a does not).  What
// a further component has (a pocket's few nodes) goes to memory lane by lane, all
// lanes at once.  At the end the workgroup's wavefronts of one component are
// added together, so a component that fills the pores gets one atomic pair per
// workgroup and not one per 64 nodes, all on one address.
constexpr int kMassThreads = 1024, kMassBlocks = 256;  // one workgroup per compute unit
constexpr int kManyLanes = 8;  // from here on one atomic pair for a component's lanes

__device__ __forceinline__ void add_sums(double *acc, int label, double x, double y) {
  unsafeAtomicAdd(acc + 2 * (int64_t)label, x);
  unsafeAtomicAdd(acc + 2 * (int64_t)label + 1, y);
}

__device__ __forceinline__ void wave_sum2(double &x, double &y) {
#pragma unroll
  for (int off = 32; off > 0; off >>= 1) {
    x += __shfl_xor(x, off);
    y += __shfl_xor(y, off);
  }
}

__global__ void __launch_bounds__(kMassThreads) k_mass(int64_t n, const int32_t *lab, int32_t count, const double *rho,
                                                       double *acc) {
  constexpr int kWaves = kMassThreads / 64;
  __shared__ int label_s[kWaves];
  __shared__ double sum_s[kWaves][2];
  int a = -1, b = -1;  // (uniform)
  double ax = 0.0, ay = 0.0, bx = 0.0, by = 0.0;
  const int lane = __lane_id(), wv = threadIdx.x >> 6;
  auto give = [&](int label, double x, double y) {  // all lanes' sums, one atomic pair
    wave_sum2(x, y);
    if (lane == 0) add_sums(acc, label, x, y);
  };
  for (int64_t base = (blockIdx.x * (int64_t)kWaves + wv) * 64; base < n; base += (int64_t)gridDim.x * kMassThreads) {
    const int64_t i = base + lane;
    const int L = i < n ? checked(lab[i], count) : -1;
    const double r = L >= 0 ? rho[i] : 0.0;
    const bool on = L >= 0, in_a = on && L == a, in_b = on && L == b;
    ax += in_a ? r : 0.0, ay += in_a ? 1.0 : 0.0;
    bx += in_b ? r : 0.0, by += in_b ? 1.0 : 0.0;
    if (__ballot(in_b) && !__ballot(in_a)) {
      std::swap(a, b);
      std::swap(ax, bx), std::swap(ay, by);
    }
    bool alone = on && !in_a && !in_b;
    int largest = 1, next = -1;
    for (uint64_t left = __ballot(alone); left;) {
      const int M = __builtin_amdgcn_readlane(L, __ffsll((unsigned long long)left) - 1);
      const uint64_t same = __ballot(L == M);
      left &= ~same;
      if (__popcll(same) > largest) largest = __popcll(same), next = M;
    }
    if (next >= 0) {
      if (a >= 0) {
        if (b >= 0) give(b, bx, by);
        b = next, bx = L == next ? r : 0.0, by = L == next ? 1.0 : 0.0;
      } else {
        a = next, ax = L == next ? r : 0.0, ay = L == next ? 1.0 : 0.0;
      }
      alone = alone && L != next;
    }
    for (uint64_t left = largest >= kManyLanes ? __ballot(alone) : 0; left;) {
      const int M = __builtin_amdgcn_readlane(L, __ffsll((unsigned long long)left) - 1);
      const uint64_t same = __ballot(L == M);
      left &= ~same;
      if (__popcll(same) < kManyLanes) continue;
      give(M, L == M ? r : 0.0, L == M ? 1.0 : 0.0);
      alone = alone && L != M;
    }
    if (alone) add_sums(acc, L, r, 1.0);
  }
  if (b >= 0) give(b, bx, by);
  wave_sum2(ax, ay);
  if (lane == 0) {
    label_s[wv] = a;
    sum_s[wv][0] = ax;
    sum_s[wv][1] = ay;
  }
  __syncthreads();
  if (wv != 0) return;
  // lane w holds wavefront w's sums; those of one component are added together
  a = lane < kWaves ? label_s[lane] : -1;
  ax = lane < kWaves ? sum_s[lane][0] : 0.0;
  ay = lane < kWaves ? sum_s[lane][1] : 0.0;
  for (uint64_t left = __ballot(a >= 0); left;) {
    const int M = __builtin_amdgcn_readlane(a, __ffsll((unsigned long long)left) - 1);
    left &= ~__ballot(a == M);
    give(M, a == M ? ax : 0.0, a == M ? ay : 0.0);
  }
}

__global__ void __launch_bounds__(kBlock) k_rescale(int64_t n, const int32_t *lab, int32_t count, const double *acc,
                                                    double rho0, double *rho) {
  const int64_t i = blockIdx.x * (int64_t)kBlock + threadIdx.x;
  if (i >= n) return;
  const int L = checked(lab[i], count);
  if (L < 0) return;
  rho[i] = rho[i] * (rho0 * acc[2 * (int64_t)L + 1] / acc[2 * (int64_t)L]);
}

struct Lattice3 {
  int32_t nx, ny, nz;
  uint32_t periodic;
};

// One sweep on bricks of 16x8x8 nodes: the brick's residuals and those of the
// nodes around it go to LDS once (0 on solid nodes, so they add nothing as
// neighbours), with a bit per node for "non-solid" in one word per x-row, and
// each thread computes four nodes from there.  With s the sum over the links
// to non-solid neighbours,
//   T r(x) = 3/2 s w c (c.r(x + c)) + 3/2 (s w c c^T) r(x):
// the first part needs no masks, the second only counts of open links.
// What bounds it: 48 LDS reads per node; 112 x 104 x 96 nodes take 28 us per
// sweep, against 58-85 us for the form that read rho, u and j of every
// neighbour from memory.
constexpr int kSx = 16, kSy = 8, kSz = 8;
constexpr int kHx = kSx + 2, kHy = kSy + 2, kHz = kSz + 2, kHaloNodes = kHx * kHy * kHz;
static_assert(kSx * kSy * kSz == 4 * kBlock && kHx <= 32, "four nodes per thread, a row's bits in one word");

// What a sweep reads and writes: the first one takes r = rho u from the
// fields; the last one writes u.
enum SweepEnds : int { kInner = 0, kFirst = 1, kLast = 2 };

// rho u, rounded once where r starts and where u is formed, so that a component
// no link carries keeps r = rho u to the end, in every bit, and comes out as 0,
// also where it is infinite or NaN (where `times` keeps it from the others)
__device__ __forceinline__ double momentum(double rho, double u) { return __dmul_rn(rho, u); }
__device__ __forceinline__ double kept(double momentum, double r) {
  return __double_as_longlong(momentum) == __double_as_longlong(r) ? 0.0 : momentum - r;
}
__device__ __forceinline__ double times(int count, double r) { return count != 0 ? count * r : 0.0; }

template <class L, int ENDS>
__global__ void __launch_bounds__(kBlock) k_link_sweep(int64_t first, Lattice3 g, const int32_t *lab, int32_t count,
                                                       const double *rho, double *u, const double *r_in,
                                                       double *r_out) {
  __shared__ double rs[3][kHaloNodes];
  __shared__ uint32_t open[kHy * kHz];
  const int64_t n = (int64_t)g.nx * g.ny * g.nz;
  const int tid = threadIdx.x;
  const int bx = (g.nx + kSx - 1) / kSx, by = (g.ny + kSy - 1) / kSy;
  const int64_t brick = first + blockIdx.x;
  const int ox = (int)(brick % bx) * kSx, oy = (int)(brick / bx % by) * kSy, oz = (int)(brick / bx / by) * kSz;
  if (tid < kHy * kHz) open[tid] = 0;
  __syncthreads();
  for (int e = tid; e < kHaloNodes; e += kBlock) {
    const int hx = e % kHx, row = e / kHx;
    int t[3] = {ox + hx - 1, oy + row % kHy - 1, oz + row / kHy - 1};
    const int ext[3] = {g.nx, g.ny, g.nz};
    bool inside = true;
    for (int a = 0; a < 3; ++a) {
      // one node beyond a face is across it or outside; further out (past a
      // ragged brick's end) is read by no node of the lattice
      const bool over = t[a] < 0 || t[a] >= ext[a];
      inside = inside && (!over || (((g.periodic >> a) & 1u) && t[a] <= ext[a]));
      if (over) t[a] = t[a] < 0 ? ext[a] - 1 : 0;
    }
    double r[3] = {0.0, 0.0, 0.0};
    const int64_t p = (int64_t)t[0] + (int64_t)g.nx * ((int64_t)t[1] + (int64_t)g.ny * t[2]);
    if (inside && checked(lab[p], count) >= 0) {
      if constexpr (ENDS & kFirst) {
        const double m = rho[p];
        for (int k = 0; k < 3; ++k) r[k] = momentum(m, u[k * n + p]);
      } else {
        for (int k = 0; k < 3; ++k) r[k] = r_in[k * n + p];
      }
      atomicOr(&open[row], 1u << hx);
    }
    for (int k = 0; k < 3; ++k) rs[k][e] = r[k];
  }
  __syncthreads();
#pragma unroll
  for (int q = 0; q < 4; ++q) {
    const int lx = tid % kSx, ly = tid / kSx % kSy, lz = tid / (kSx * kSy) + q * (kSz / 4);
    const int x = ox + lx, y = oy + ly, z = oz + lz;
    if (x >= g.nx || y >= g.ny || z >= g.nz) continue;
    const int c0 = lx + 1 + kHx * (ly + 1 + kHy * (lz + 1)), row0 = ly + 1 + kHy * (lz + 1);
    const int64_t i = (int64_t)x + (int64_t)g.nx * ((int64_t)y + (int64_t)g.ny * z);
    if (!((open[row0] >> (lx + 1)) & 1u)) {
      if constexpr (!(ENDS & kLast))
        for (int k = 0; k < 3; ++k) r_out[k * n + i] = 0.0;
      continue;
    }
    const double r0[3] = {rs[0][c0], rs[1][c0], rs[2][c0]};
    const bool finite = __builtin_isfinite(r0[0]) && __builtin_isfinite(r0[1]) && __builtin_isfinite(r0[2]);
    double acc[3] = {0.0, 0.0, 0.0};  // 2/3 T r, weight by weight
    lbm::static_for<2>([&](auto Cls) {
      constexpr bool edge = decltype(Cls)::value == 1;  // links with two nonzero components, or one
      double s[3] = {0.0, 0.0, 0.0};
      int diag[3] = {0, 0, 0}, off[3] = {0, 0, 0};  // counts of c_a c_a, and of c_a c_b for ab = yz, xz, xy
      lbm::static_for<L::Q>([&](auto d) {
        constexpr int cx = L::C[d][0], cy = L::C[d][1], cz = L::C[d][2];
        constexpr int nz = (cx != 0) + (cy != 0) + (cz != 0);
        if constexpr (nz == (edge ? 2 : 1)) {
          const int t = c0 + cx + kHx * (cy + kHy * cz);
          double v = 0.0;
          if constexpr (cx != 0) v += cx * rs[0][t];
          if constexpr (cy != 0) v += cy * rs[1][t];
          if constexpr (cz != 0) v += cz * rs[2][t];
          if constexpr (cx != 0) s[0] += cx * v;
          if constexpr (cy != 0) s[1] += cy * v;
          if constexpr (cz != 0) s[2] += cz * v;
          const int b = (int)((open[row0 + cy + kHy * cz] >> (lx + 1 + cx)) & 1u);
          if constexpr (cx != 0) diag[0] += b;
          if constexpr (cy != 0) diag[1] += b;
          if constexpr (cz != 0) diag[2] += b;
          if constexpr (cy * cz != 0) off[0] += cy * cz * b;
          if constexpr (cx * cz != 0) off[1] += cx * cz * b;
          if constexpr (cx * cy != 0) off[2] += cx * cy * b;
        }
      });
      if (finite) {
        s[0] += diag[0] * r0[0] + off[2] * r0[1] + off[1] * r0[2];
        s[1] += off[2] * r0[0] + diag[1] * r0[1] + off[0] * r0[2];
        s[2] += off[1] * r0[0] + off[0] * r0[1] + diag[2] * r0[2];
      } else {
        s[0] += times(diag[0], r0[0]) + times(off[2], r0[1]) + times(off[1], r0[2]);
        s[1] += times(off[2], r0[0]) + times(diag[1], r0[1]) + times(off[0], r0[2]);
        s[2] += times(off[1], r0[0]) + times(off[0], r0[1]) + times(diag[2], r0[2]);
      }
      constexpr double w = 1.5 * L::Wt[edge ? L::Q - 1 : 1];
      for (int k = 0; k < 3; ++k) acc[k] += w * s[k];
    });
    if constexpr (ENDS & kLast) {
      const double m = rho[i];
      for (int k = 0; k < 3; ++k) u[k * n + i] = kept(momentum(m, u[k * n + i]), r0[k] - acc[k]) / m;
    } else {
      for (int k = 0; k < 3; ++k) r_out[k * n + i] = r0[k] - acc[k];
    }
  }
}

// u = (rho u - r) / rho after a single sweep (which reads its neighbours' u)
__global__ void __launch_bounds__(kBlock) k_velocity(int64_t n, const int32_t *lab, int32_t count, const double *rho,
                                                     const double *r, double *u) {
  const int64_t i = blockIdx.x * (int64_t)kBlock + threadIdx.x;
  if (i >= n || checked(lab[i], count) < 0) return;
  const double m = rho[i];
  for (int k = 0; k < 3; ++k) u[k * n + i] = kept(momentum(m, u[k * n + i]), r[k * n + i]) / m;
}

template <class L>
void launch_sweeps(int64_t n, Lattice3 g, const int32_t *labels, int32_t count, const double *rho, double *u,
                   double *ra, double *rb, int iterations, hipStream_t s) {
  const int64_t bricks =
      (int64_t)((g.nx + kSx - 1) / kSx) * ((g.ny + kSy - 1) / kSy) * ((g.nz + kSz - 1) / kSz);
  auto sweep = [&](auto ends, const double *r_in, double *r_out) {
    // as many launches as threads per launch ask for (flat lattices of 2^31 nodes: two)
    constexpr int64_t most = UINT32_MAX / kBlock;
    for (int64_t first = 0; first < bricks; first += most)
      hipLaunchKernelGGL((k_link_sweep<L, decltype(ends)::value>), dim3((unsigned)std::min(most, bricks - first)),
                         dim3(kBlock), 0, s, first, g, labels, count, rho, u, r_in, r_out);
  };
  sweep(std::integral_constant<int, kFirst>{}, nullptr, ra);
  if (iterations == 1) {
    hipLaunchKernelGGL(k_velocity, dim3((unsigned)((n + kBlock - 1) / kBlock)), dim3(kBlock), 0, s, n, labels, count,
                       rho, (const double *)ra, u);
    return;
  }
  for (int it = 1; it + 1 < iterations; ++it) {
    sweep(std::integral_constant<int, kInner>{}, ra, rb);
    std::swap(ra, rb);
  }
  sweep(std::integral_constant<int, kLast>{}, ra, rb);
}

}  // namespace

extern "C" int lbm_project_invariants(int32_t q, const int32_t shape[3], uint32_t periodic, const int32_t *labels,
                                      int32_t count, double rho0, int32_t iterations, double *rho, double *u,
                                      double *scratch, void *stream) {
  if (!shape || !labels || !rho || !u || !scratch)
    return set_error(LBM_ERR_ARG, "lbm_project_invariants: NULL argument");
  if (q != 9 && q != 19) return set_error(LBM_ERR_UNSUPPORTED, "lbm_project_invariants: q = %d", q);
  if (shape[0] <= 0 || shape[1] <= 0 || shape[2] <= 0 || (q == 9 && shape[2] != 1))
    return set_error(LBM_ERR_ARG, "lbm_project_invariants: shape %d x %d x %d for q = %d", shape[0], shape[1],
                     shape[2], q);
  if (periodic > 7u) return set_error(LBM_ERR_ARG, "lbm_project_invariants: periodic bits %u", periodic);
  if (!(rho0 > 0.0) || rho0 > 1e300) return set_error(LBM_ERR_ARG, "lbm_project_invariants: rho0 = %g", rho0);
  if (iterations < 1 || iterations > kMaxIterations)
    return set_error(LBM_ERR_ARG, "lbm_project_invariants: iterations = %d (1..%d)", iterations, kMaxIterations);
  const int64_t n = (int64_t)shape[0] * shape[1] * shape[2];
  if (count < 0 || count > n)
    return set_error(LBM_ERR_ARG, "lbm_project_invariants: count = %d for %lld nodes", count, (long long)n);
  if (count == 0) return LBM_OK;  // no non-solid node
  hipStream_t s = (hipStream_t)stream;
  const unsigned grid = (unsigned)((n + kBlock - 1) / kBlock);
  const int64_t sums = 2 * (int64_t)count;
  const unsigned clear_grid = (unsigned)std::min<int64_t>((sums + kBlock - 1) / kBlock, 4096);
  double *acc = scratch;
  double *ra = scratch + sums, *rb = ra + 3 * n;
  hipLaunchKernelGGL(k_clear, dim3(clear_grid), dim3(kBlock), 0, s, acc, sums);
  const int64_t mass_blocks = std::min<int64_t>((n + kMassThreads - 1) / kMassThreads, kMassBlocks);
  hipLaunchKernelGGL(k_mass, dim3((unsigned)mass_blocks), dim3(kMassThreads), 0, s, n, labels, count,
                     (const double *)rho, acc);
  hipLaunchKernelGGL(k_rescale, dim3(grid), dim3(kBlock), 0, s, n, labels, count, (const double *)acc, rho0, rho);
  const Lattice3 g{shape[0], shape[1], shape[2], periodic};
  if (q == 19)
    launch_sweeps<lbm::D3Q19>(n, g, labels, count, rho, u, ra, rb, iterations, s);
  else
    launch_sweeps<lbm::D2Q9>(n, g, labels, count, rho, u, ra, rb, iterations, s);
  const hipError_t e = hipGetLastError();
  if (e != hipSuccess) return set_error(LBM_ERR_HIP, "lbm_project_invariants: %s", hipGetErrorString(e));
  return LBM_OK;
}

// ---- connected components on the device ---------------------------------------
// The same labels as the host lbm_components, for a warm start that must
// not wait for the host.  Lock-free union-find over the links: every
// pointer goes from a node to a node of smaller index, a union hooks the
// larger of two roots under the smaller with a compare-and-swap (retrying
// from the new parent if the root moved meanwhile), and finds halve their
// paths.  Because every parent index is smaller than its node's, every loop
// ends: a find walks strictly decreasing indices and a failed hook lowers
// the larger root.  The root of a component is then its smallest node, so
// numbering roots in scan order (an exclusive prefix sum of root flags)
// reproduces the host's numbering by first appearance.
namespace {

constexpr int kScanBlock = 1024;  // threads of the scan kernels
constexpr int kScanItems = 4;     // items per thread

__device__ __forceinline__ int32_t ld_parent(const int32_t *p) {
  return __hip_atomic_load(p, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT);
}

__device__ __forceinline__ int32_t cc_find(int32_t *parent, int32_t v) {
  while (true) {
    const int32_t p = ld_parent(parent + v);
    if (p == v) return v;
    const int32_t gp = ld_parent(parent + p);
    if (gp == p) return p;
    __hip_atomic_store(parent + v, gp, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT);  // an ancestor of v
    v = gp;
  }
}

__global__ void __launch_bounds__(kBlock) k_cc_init(int64_t n, const uint8_t *solid, int32_t *parent) {
  for (int64_t e = (int64_t)blockIdx.x * kBlock + threadIdx.x; e < n; e += (int64_t)gridDim.x * kBlock)
    parent[e] = solid[e] ? -1 : (int32_t)e;
}

struct CcGrid {
  int nx, ny, nz;
};

// Joins the trees of nodes e and f.
__device__ __forceinline__ void cc_join(int32_t *parent, int32_t e, int32_t f) {
  int32_t a = cc_find(parent, e), b = cc_find(parent, f);
  while (a != b) {
    if (a > b) {
      const int32_t s = a;
      a = b;
      b = s;
    }
    const int32_t old = atomicCAS(parent + b, b, a);
    if (old == b) break;  // b now hangs under a
    b = cc_find(parent, old);
    a = cc_find(parent, a);
  }
}

// The node one link c away from (x, y, z), or -1 past an edge that does not wrap.
__device__ __forceinline__ int64_t cc_link(const CcGrid &g, uint32_t periodic, int x, int y, int z, int cx, int cy,
                                           int cz) {
  int t[3] = {x + cx, y + cy, z + cz};
  const int ext[3] = {g.nx, g.ny, g.nz};
  for (int a = 0; a < 3; ++a) {
    if (t[a] >= 0 && t[a] < ext[a]) continue;
    if (!((periodic >> a) & 1u)) return -1;
    t[a] = t[a] < 0 ? t[a] + ext[a] : t[a] - ext[a];
  }
  return (int64_t)t[0] + (int64_t)g.nx * ((int64_t)t[1] + (int64_t)g.ny * t[2]);
}

// One thread per node: union with the non-solid node one link away, for one
// link of each opposite pair, only links with c_axis != 0.
template <class L>
__global__ void __launch_bounds__(kBlock) k_cc_union(CcGrid g, uint32_t periodic, int axis, const uint8_t *solid,
                                                     int32_t *parent) {
  const int64_t n = (int64_t)g.nx * g.ny * g.nz;
  const int64_t e = (int64_t)blockIdx.x * kBlock + threadIdx.x;
  if (e >= n || solid[e]) return;
  const int x = (int)(e % g.nx), y = (int)((e / g.nx) % g.ny), z = (int)(e / ((int64_t)g.nx * g.ny));
  lbm::static_for<L::Q>([&](auto I) {
    constexpr int i = decltype(I)::value;
    constexpr int cx = L::C[i][0], cy = L::C[i][1], cz = L::C[i][2];
    if constexpr ((cx != 0 || cy != 0 || cz != 0) && i < L::Opp[i]) {
      if ((axis == 0 ? cx : axis == 1 ? cy : cz) == 0) return;
      const int64_t f = cc_link(g, periodic, x, y, z, cx, cy, cz);
      if (f >= 0 && !solid[f]) cc_join(parent, (int32_t)e, (int32_t)f);
    }
  });
}

// With every link (axis = -1) most unions say what others already do, so the
// links are thinned first.  k_cc_runs hangs each node under the first node of
// its x-run inside its wavefront's 64 nodes (one ballot, no search).  Then
//   - an x-link joins only where a run crosses a wavefront's start or wraps;
//   - a link with c_x = 0 whose copy one node to the left exists is implied by
//     it (both ends are joined to their left neighbours by x-links);
//   - a diagonal link is implied where either of its two corners is non-solid.
// 128^3 at porosity 0.5: 530-600 us for nine unions per node, 134-144 us so.
__global__ void __launch_bounds__(kBlock) k_cc_runs(CcGrid g, const uint8_t *solid, int32_t *parent) {
  const int64_t n = (int64_t)g.nx * g.ny * g.nz;
  const int64_t e = (int64_t)blockIdx.x * kBlock + threadIdx.x;
  const bool fluid = e < n && !solid[e];
  const uint64_t open = __ballot(fluid), edge = __ballot(e % g.nx == 0);
  const uint64_t starts = open & (~(open << 1) | edge);  // (lane 0: nothing to its left in this wavefront)
  if (e >= n) return;
  const int lane = __lane_id();
  const int first = 63 - __clzll((long long)(starts & (~0ull >> (63 - lane))));
  parent[e] = fluid ? (int32_t)(e - lane + first) : -1;
}

template <class L>
__global__ void __launch_bounds__(kBlock) k_cc_union_all(CcGrid g, uint32_t periodic, const uint8_t *solid,
                                                         int32_t *parent) {
  const int64_t n = (int64_t)g.nx * g.ny * g.nz;
  const int64_t e = (int64_t)blockIdx.x * kBlock + threadIdx.x;
  if (e >= n || solid[e]) return;
  const int x = (int)(e % g.nx), y = (int)((e / g.nx) % g.ny), z = (int)(e / ((int64_t)g.nx * g.ny));
  const bool left = x > 0 && !solid[e - 1];
  auto open = [&](int cx, int cy, int cz) {
    const int64_t f = cc_link(g, periodic, x, y, z, cx, cy, cz);
    return f >= 0 && !solid[f];
  };
  lbm::static_for<L::Q>([&](auto I) {
    constexpr int i = decltype(I)::value;
    constexpr int cx = L::C[i][0], cy = L::C[i][1], cz = L::C[i][2];
    if constexpr ((cx != 0 || cy != 0 || cz != 0) && i < L::Opp[i]) {
      if constexpr (cx != 0 && cy == 0 && cz == 0)
        if (x + 1 < g.nx && ((e + 1) & 63) != 0) return;  // one run of one wavefront
      const int64_t f = cc_link(g, periodic, x, y, z, cx, cy, cz);
      if (f < 0 || solid[f]) return;
      if constexpr (cx == 0)
        if (left && !solid[f - 1]) return;
      if constexpr ((cx != 0) + (cy != 0) + (cz != 0) == 2) {
        if (open(cx, cx != 0 ? 0 : cy, 0)) return;
        if (open(0, cx != 0 ? cy : 0, cz)) return;
      }
      cc_join(parent, (int32_t)e, (int32_t)f);
    }
  });
}

// parent <- root; flag = 1 on roots (in the scan buffer).  The walk to the
// root only reads: the single write per node is its root, so a concurrent
// walk through that node sees an ancestor either way, and every node ends
// holding its root.
__global__ void __launch_bounds__(kBlock) k_cc_flatten(int64_t n, int32_t *parent, int32_t *flag) {
  for (int64_t e = (int64_t)blockIdx.x * kBlock + threadIdx.x; e < n; e += (int64_t)gridDim.x * kBlock) {
    const int32_t p = parent[e];
    if (p < 0) {
      flag[e] = 0;
      continue;
    }
    int32_t r = (int32_t)e;
    for (int32_t up = p; up != r; up = ld_parent(parent + up)) r = up;
    flag[e] = r == (int32_t)e;
    __hip_atomic_store(parent + e, r, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT);
  }
}

// Exclusive prefix sum of v[0, n) in place, kScanBlock * kScanItems items per
// block; the block totals go to sums[blockIdx.x].
__global__ void __launch_bounds__(kScanBlock) k_scan_block(int64_t n, int32_t *v, int32_t *sums) {
  __shared__ int32_t s[kScanBlock];
  const int64_t base = ((int64_t)blockIdx.x * kScanBlock + threadIdx.x) * kScanItems;
  int32_t item[kScanItems], run = 0;
  for (int k = 0; k < kScanItems; ++k) {
    item[k] = base + k < n ? v[base + k] : 0;
    run += item[k];
  }
  s[threadIdx.x] = run;
  __syncthreads();
  for (int off = 1; off < kScanBlock; off <<= 1) {  // inclusive Hillis-Steele scan of the thread totals
    const int32_t t = threadIdx.x >= (unsigned)off ? s[threadIdx.x - off] : 0;
    __syncthreads();
    s[threadIdx.x] += t;
    __syncthreads();
  }
  int32_t acc = s[threadIdx.x] - run;
  for (int k = 0; k < kScanItems; ++k) {
    if (base + k < n) v[base + k] = acc;
    acc += item[k];
  }
  if (threadIdx.x == kScanBlock - 1) sums[blockIdx.x] = s[threadIdx.x];
}

// Exclusive scan of the block totals (one block, any count); total to sums[nb].
__global__ void __launch_bounds__(kScanBlock) k_scan_sums(int64_t nb, int32_t *sums) {
  __shared__ int32_t s[kScanBlock];
  int32_t carry = 0;
  for (int64_t b0 = 0; b0 < nb; b0 += kScanBlock) {
    const int64_t b = b0 + threadIdx.x;
    const int32_t x = b < nb ? sums[b] : 0;
    s[threadIdx.x] = x;
    __syncthreads();
    for (int off = 1; off < kScanBlock; off <<= 1) {
      const int32_t t = threadIdx.x >= (unsigned)off ? s[threadIdx.x - off] : 0;
      __syncthreads();
      s[threadIdx.x] += t;
      __syncthreads();
    }
    if (b < nb) sums[b] = carry + s[threadIdx.x] - x;
    const int32_t total = s[kScanBlock - 1];
    __syncthreads();
    carry += total;
  }
  if (threadIdx.x == 0) sums[nb] = carry;
}

// labels = rank of the node's root among the roots (the root's flag slot
// holds it once offset by its block's total); -1 on solid nodes
__global__ void __launch_bounds__(kBlock) k_cc_label(int64_t n, const int32_t *rank, const int32_t *sums,
                                                     int32_t *parent_to_label) {
  constexpr int64_t per = (int64_t)kScanBlock * kScanItems;
  for (int64_t e = (int64_t)blockIdx.x * kBlock + threadIdx.x; e < n; e += (int64_t)gridDim.x * kBlock) {
    const int32_t r = parent_to_label[e];
    parent_to_label[e] = r < 0 ? -1 : rank[r] + sums[r / per];
  }
}

unsigned cc_grid(int64_t n) {
  const int64_t b = (n + kBlock - 1) / kBlock;
  return (unsigned)(b < 16384 ? (b > 0 ? b : 1) : 16384);
}

}  // namespace

extern "C" int64_t lbm_components_device_scratch(const int32_t shape[3]) {
  if (!shape || shape[0] <= 0 || shape[1] <= 0 || shape[2] <= 0) return -1;
  const int64_t n = (int64_t)shape[0] * shape[1] * shape[2];
  const int64_t per = (int64_t)kScanBlock * kScanItems;
  return n + (n + per - 1) / per + 1;
}

namespace {

// The labelling behind both device entry points; scratch holds
// lbm_components_device_scratch(shape) int32 entries, every one written
// before it is read.
int components_device(const char *who, int32_t q, const uint8_t *solid, const int32_t shape[3], uint32_t periodic,
                      int32_t axis, int32_t *labels, int32_t *count, int32_t *scratch, hipStream_t s) {
  const int64_t n = (int64_t)shape[0] * shape[1] * shape[2];
  const CcGrid g{shape[0], shape[1], shape[2]};
  const int64_t per = (int64_t)kScanBlock * kScanItems, nb = (n + per - 1) / per;
  int32_t *flag = scratch, *sums = scratch + n;
  const unsigned all = (unsigned)((n + kBlock - 1) / kBlock);
  if (axis < 0) {
    hipLaunchKernelGGL(k_cc_runs, dim3(all), dim3(kBlock), 0, s, g, solid, labels);
    if (q == 19)
      hipLaunchKernelGGL(k_cc_union_all<lbm::D3Q19>, dim3(all), dim3(kBlock), 0, s, g, periodic, solid, labels);
    else
      hipLaunchKernelGGL(k_cc_union_all<lbm::D2Q9>, dim3(all), dim3(kBlock), 0, s, g, periodic, solid, labels);
  } else {
    hipLaunchKernelGGL(k_cc_init, dim3(cc_grid(n)), dim3(kBlock), 0, s, n, solid, labels);
    if (q == 19)
      hipLaunchKernelGGL(k_cc_union<lbm::D3Q19>, dim3(all), dim3(kBlock), 0, s, g, periodic, axis, solid, labels);
    else
      hipLaunchKernelGGL(k_cc_union<lbm::D2Q9>, dim3(all), dim3(kBlock), 0, s, g, periodic, axis, solid, labels);
  }
  hipLaunchKernelGGL(k_cc_flatten, dim3(cc_grid(n)), dim3(kBlock), 0, s, n, labels, flag);
  hipLaunchKernelGGL(k_scan_block, dim3((unsigned)nb), dim3(kScanBlock), 0, s, n, flag, sums);
  hipLaunchKernelGGL(k_scan_sums, dim3(1), dim3(kScanBlock), 0, s, nb, sums);
  hipLaunchKernelGGL(k_cc_label, dim3(cc_grid(n)), dim3(kBlock), 0, s, n, flag, sums, labels);
  hipError_t e = hipGetLastError();
  if (e == hipSuccess) e = hipMemcpyAsync(count, sums + nb, sizeof(int32_t), hipMemcpyDeviceToHost, s);
  if (e == hipSuccess) e = hipStreamSynchronize(s);
  if (e != hipSuccess) return set_error(LBM_ERR_HIP, "%s: %s", who, hipGetErrorString(e));
  return LBM_OK;
}

// Argument checks shared by both device entry points.
int components_device_args(const char *who, int32_t q, const uint8_t *solid, const int32_t shape[3],
                           uint32_t periodic, int32_t axis, const int32_t *labels, const int32_t *count) {
  if (!solid || !shape || !labels || !count) return set_error(LBM_ERR_ARG, "%s: NULL argument", who);
  if (q != 9 && q != 19) return set_error(LBM_ERR_UNSUPPORTED, "%s: q = %d", who, q);
  if (shape[0] <= 0 || shape[1] <= 0 || shape[2] <= 0)
    return set_error(LBM_ERR_ARG, "%s: shape %d x %d x %d", who, shape[0], shape[1], shape[2]);
  if (q == 9 && shape[2] != 1) return set_error(LBM_ERR_ARG, "%s: D2Q9 needs shape[2] = 1", who);
  if (periodic > 7u) return set_error(LBM_ERR_ARG, "%s: periodic bits %u", who, periodic);
  if (axis < -1 || axis >= (q == 9 ? 2 : 3)) return set_error(LBM_ERR_ARG, "%s: axis %d for q = %d", who, axis, q);
  const int64_t n = (int64_t)shape[0] * shape[1] * shape[2];
  if (n > INT32_MAX) return set_error(LBM_ERR_ARG, "%s: %lld nodes exceed int32 labels", who, (long long)n);
  return LBM_OK;
}

// Fixed scratch of lbm_components_device_noalloc: one copy per GPU, held
// until the process ends.  Host code never passes this name to a kernel (on
// the host it is only a stand-in for the symbol); it uses the device address
// hipGetSymbolAddress returns for the current device.
constexpr int64_t kNoAllocEntries = int64_t(1) << 22;  // int32 entries, 16 MiB
static __device__ __align__(256) int32_t cc_noalloc_scratch[kNoAllocEntries];

constexpr int kMaxDevices = 64;

// Device address of cc_noalloc_scratch on the current device, looked up
// once per device (with that device current) and kept.
int noalloc_scratch(const char *who, int32_t **out) {
  static std::mutex mu;
  static int32_t *addr[kMaxDevices] = {};
  int dev = 0;
  hipError_t e = hipGetDevice(&dev);
  if (e != hipSuccess) return set_error(LBM_ERR_HIP, "%s: %s", who, hipGetErrorString(e));
  if (dev < 0 || dev >= kMaxDevices) return set_error(LBM_ERR_UNSUPPORTED, "%s: device %d", who, dev);
  std::lock_guard<std::mutex> lock(mu);
  if (!addr[dev]) {
    void *p = nullptr;
    e = hipGetSymbolAddress(&p, HIP_SYMBOL(cc_noalloc_scratch));
    if (e != hipSuccess || !p)
      return set_error(LBM_ERR_HIP, "%s: scratch address: %s", who, hipGetErrorString(e));
    addr[dev] = static_cast<int32_t *>(p);
  }
  *out = addr[dev];
  return LBM_OK;
}

}  // namespace

extern "C" int lbm_components_device(int32_t q, const uint8_t *solid, const int32_t shape[3], uint32_t periodic,
                                     int32_t axis, int32_t *labels, int32_t *count, int32_t *scratch,
                                     void *stream) {
  const char *who = "lbm_components_device";
  if (!scratch) return set_error(LBM_ERR_ARG, "%s: NULL argument", who);
  const int r = components_device_args(who, q, solid, shape, periodic, axis, labels, count);
  if (r != LBM_OK) return r;
  return components_device(who, q, solid, shape, periodic, axis, labels, count, scratch,
                           static_cast<hipStream_t>(stream));
}

extern "C" int64_t lbm_components_noalloc_max_scratch(void) { return kNoAllocEntries; }

extern "C" int lbm_components_device_noalloc(int32_t q, const uint8_t *solid, const int32_t shape[3],
                                             uint32_t periodic, int32_t axis, int32_t *labels, int32_t *count,
                                             void *stream) {
  const char *who = "lbm_components_device_noalloc";
  const int r = components_device_args(who, q, solid, shape, periodic, axis, labels, count);
  if (r != LBM_OK) return r;
  const int64_t need = lbm_components_device_scratch(shape);
  if (need > kNoAllocEntries)
    return set_error(LBM_ERR_ARG, "%s: %d x %d x %d needs %lld scratch entries, above the fixed %lld", who, shape[0],
                     shape[1], shape[2], (long long)need, (long long)kNoAllocEntries);
  int32_t *scratch = nullptr;
  const int e = noalloc_scratch(who, &scratch);
  if (e != LBM_OK) return e;
  return components_device(who, q, solid, shape, periodic, axis, labels, count, scratch,
                           static_cast<hipStream_t>(stream));
}
