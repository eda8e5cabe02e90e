// D2Q9 steps on 16x16 tiles, several per launch.
//
// A workgroup takes a window of 32x32 nodes, one per thread, reads its
// post-collision PDFs once, and runs K steps there: each step exchanges the
// nodes' values through LDS (a non-solid source's f*_i(x - c_i), or the node's
// own f*_opp(i) on a half-way bounce-back) and collides in registers.  What the
// window's edge lacks makes one more layer wrong per step, so after K steps the
// inner (32 - 2K)^2 nodes are those of K single steps, bit for bit, and are
// written; the layers around are computed again by the neighbouring windows.
// So a launch moves each PDF once in and once out for K steps, and a grid too
// small to fill the device pays one launch for K steps.
//
// What bounds it: vector arithmetic at two workgroups per compute unit (FP64: one thread
// per node, 64 registers) and, where a window's nodes are read, HBM: 1.78 reads
// and one write of each PDF per four steps.  What is the same for all nodes is
// kept in scalar registers (uniform()): without that FP64 needs 82 vector
// registers, runs one workgroup per compute unit and spills if it is held to 64
// (a fifth to nearly a half slower on the 1536x1500 channel with discs).
// Per step, k_step before -> this: that channel 39.7 -> 33.3 us (FP64), 27.2 ->
// 21.0 (FP32); the sweep over sizes and steps per launch stands at steps9_runs.
//
// Steps of other forms (one PDF copy, a lid, FP16 storage, which rounds every
// step to 16 bits, batches) and single steps run k_step (kernels.hip).
#include <algorithm>

#include "device.h"
#include "kernels.h"

namespace lbm {
namespace {

constexpr int kWin = 32, kThreads = kWin * kWin;   // window edge, threads
constexpr int kMostSteps = 10;                     // per launch
constexpr int kPitch = kWin + 2, kArea = kPitch * kPitch;  // with a guard ring

struct Window {
  int nx, ny, tgx, periodic;
  int steps, wx;  // steps of this launch; windows along x
};

template <int S, bool INC, bool MRT>
__global__ void __launch_bounds__(kThreads, (S == LBM_F64 && MRT ? 4 : 8))
    k_steps9(const void *__restrict__ src_, void *__restrict__ dst_, TileArgs a, const int32_t *__restrict__ tmap,
             Window w, double omega) {
  using L = D2Q9;
  using St = Store<S>;
  using T = typename St::T;
  using R = typename St::R;
  constexpr int Q = L::Q, AX = 16, W = 4;
  extern __shared__ __attribute__((aligned(16))) char lds[];
  R *const x8 = reinterpret_cast<R *>(lds);                      // [8][kArea]: direction i at (i - 1) kArea
  uint8_t *const open_s = reinterpret_cast<uint8_t *>(x8 + 8 * kArea);  // [kArea]
  const T *src = static_cast<const T *>(src_);
  T *dst = static_cast<T *>(dst_);
  const int tid = threadIdx.x, lx = tid % kWin, ly = tid / kWin;
  const int at = (lx + 1) + kPitch * (ly + 1);
  const int out = kWin - 2 * w.steps;  // edge of the window's result
  const int blk = (int)xcd_remap(blockIdx.x, gridDim.x);
  const int px = blk % w.wx * out + lx - w.steps, py = blk / w.wx * out + ly - w.steps;
  auto wrap = [](int v, int n, bool periodic) -> int {  // -1 past a wall
    if (v >= 0 && v < n) return v;
    if (!periodic) return -1;
    v %= n;
    return v < 0 ? v + n : v;
  };
  const int x = wrap(px, w.nx, w.periodic & 1), y = wrap(py, w.ny, w.periodic & 2);
  bool fluid = false;
  int64_t entry = 0;
  int n = 0;
  if (x >= 0 && y >= 0) {
    const int32_t tile = tmap[x / AX + w.tgx * (y / AX)];
    if (tile >= 0) {
      const int ell = x % AX + AX * (y % AX), wd = ell >> 6, b = ell & 63;
      const uint64_t m = a.fluid[(int64_t)tile * W + wd];
      if ((m >> b) & 1ull) {
        const TileRec r = a.rec[tile];
        fluid = true;
        n = r.n;
        entry = r.off + a.pre[(int64_t)tile * W + wd] + __popcll(m & ((1ull << b) - 1ull));
      }
    }
  }
  for (int k = tid; k < kArea; k += kThreads) open_s[k] = 0;
  if (!__syncthreads_or(fluid)) return;  // nothing but solid nodes in this window
  open_s[at] = fluid;
  R f[Q];
  static_for<Q>([&](auto I) {
    constexpr int i = decltype(I)::value;
    f[i] = fluid ? St::load(src, entry + (int64_t)i * n, a.f16_inv) : R(0);
  });
  __syncthreads();
  uint32_t open = 0;  // bit i: the source of direction i is non-solid
  static_for<Q>([&](auto I) {
    constexpr int i = decltype(I)::value;
    if (i > 0 && open_s[at - L::C[i][0] - kPitch * L::C[i][1]]) open |= 1u << i;
  });
  const R gx = (R)a.samples[0].g[0], gy = (R)a.samples[0].g[1], gz = (R)a.samples[0].g[2];
  const BgkRate<L, R> rate = uniform(bgk_rate<L>((R)omega, gx, gy, gz));
  for (int t = 0; t < w.steps; ++t) {
    if (fluid)
      static_for<Q - 1>([&](auto I) {
        constexpr int i = decltype(I)::value + 1;
        x8[(i - 1) * kArea + at] = f[i];
      });
    __syncthreads();
    R g[Q];
    g[0] = f[0];
    static_for<Q - 1>([&](auto I) {
      constexpr int i = decltype(I)::value + 1;
      const R v = x8[(i - 1) * kArea + at - L::C[i][0] - kPitch * L::C[i][1]];
      g[i] = (open >> i) & 1u ? v : f[L::Opp[i]];
    });
    __syncthreads();  // every value of this step is read
    R sum, jx, jy, jz;
    moment_sums<L>(g, sum, jx, jy, jz);
    if constexpr (MRT)
      collide_mrt<L, S, INC>(g, sum, jx, jy, jz, (R)a.rho0, gx, gy, gz, a.mrt);
    else
      collide_bgk<L, S, INC>(g, sum, jx, jy, jz, (R)a.rho0, rate);
    static_for<Q>([&](auto I) { f[decltype(I)::value] = g[decltype(I)::value]; });
  }
  const bool inner = lx >= w.steps && lx < kWin - w.steps && ly >= w.steps && ly < kWin - w.steps;
  if (fluid && inner && px < w.nx && py < w.ny)  // (an inner node's px, py are not negative)
    static_for<Q>([&](auto I) {
      constexpr int i = decltype(I)::value;
      St::store(dst, entry + (int64_t)i * n, f[i], a.f16_scale);
    });
}

int windows(int n, int steps) { return (n - 1) / (kWin - 2 * steps) + 1; }

}  // namespace

// How n steps are launched.
//
// Where the windows of four steps are no more than the compute units, all run
// at once and a launch costs its latency: as many steps per launch as leave it
// so, ten at most.  Else four, where the doubled layers weigh less.  One sweep
// over the steps per launch, us per step by 1, 2, 3, 4, 5, 6, 8, 10:
//   64x64      FP64  4.0  4.3  3.4  2.8  2.6  2.4  2.1  2.0
//              FP32  3.9  3.9  2.9  2.2  2.1  1.9  1.7  1.6
//   256x256    FP64  4.3  4.6  3.5  3.0  2.7  2.5  2.2  3.2   (256 windows by 8, 484 by 10)
//              FP32  4.1  4.0  3.0  2.3  2.3  2.0  1.7  2.4
//   320x320    FP64  5.1  4.7  3.6  3.1  2.8  2.5  3.4  4.6   (256 by 6, 324 by 7)
//   384x384    FP64  5.9  4.8  3.7  3.0  4.1  3.8  5.0  5.9   (256 by 4, 324 by 5)
//   512x512    FP64  7.3  7.6  5.9  4.9  6.1  5.7  6.4  11
//              FP32  5.8  5.8  4.1  3.4  4.5  4.1  4.5  7.7
//   1500x1536  FP64  36.4 37.3 34.3 32.8 34.8 38.2 53   86
//              FP32  25.4 27.4 22.8 20.7 22.8 25.2 35   57
//   4096x4096  FP64  303  312  281  267  266  279  376  623
//              FP32  214  223  173  150  166  180  249  417
// so FP32 takes the same numbers as FP64, and launches of two steps alone do not pay.
// MRT, whose FP64 form does not fit 64 registers, gains on small grids only:
//   64x64      FP64  4.3  4.8  3.9  3.4  3.2  3.0  2.7  2.6
//   384x384    FP64  6.2  5.3  4.3  3.7  6.1  5.8  7.8  9.9
//   1500x1536  FP64  40.2 52.1 49.2 48.9;  FP32  27.7 35.0 31.2 29.6
//
// The launches are as many as n modulo 2, so that n steps leave the state in
// the copy where n single steps leave it: a caller that captured an even
// number of steps replays them from the copy they end in.  A launch of an odd
// number of steps keeps to that by itself, one of an even number comes with
// another: `most` steps in pairs of launches (if it is even), then for the rest
// one or two launches and one or two single steps (50 steps by four: twelve
// launches and two single steps, 32.9 us per step at 1536x1500 FP64; spread
// evenly over fourteen launches 33.3).
//
// Single steps alone stay for geometries with fewer than one tile for every four
// windows, where most of a launch would look at solid nodes, and where the grid
// would not fit a launch.
StepRuns steps9_runs(const Variant &v, const int32_t shape[3], int64_t n_waves, int n) {
  const StepRuns single{{{1, n}, {0, 0}, {0, 0}}};
  if (v.q != 9 || v.storage == LBM_F16_OFFSET || shape[2] != 1 || n < 3) return single;
  auto grid = [&](int k) { return (int64_t)windows(shape[0], k) * windows(shape[1], k); };
  constexpr int kUnits = 256;
  const bool small = grid(4) <= kUnits;
  if (!small && v.collision == LBM_COLLISION_MRT) return single;
  int most = 4;
  while (small && most < kMostSteps && grid(most + 1) <= std::min<int64_t>(kUnits, n_waves)) ++most;
  const int pair = most % 2 ? 1 : 2, full = n / (pair * most) * pair, r = n - full * most;
  StepRuns p{{{most, full}, {0, 0}, {1, r}}};
  auto rest = [&](int steps, int launches) {
    p.run[1] = {steps, launches};
    p.run[2].launches = r - steps * launches;
  };
  if (r > most + 1 && r / 2 >= 3)
    rest(r / 2, 2);  // (and a single step if r is odd)
  else if (r >= 3)
    rest(r % 2 ? std::min(r, most - (most % 2 ? 0 : 1)) : r - 1, 1);  // odd
  const int64_t blocks = grid(full ? most : p.run[1].steps);
  return p.run[0].launches + p.run[1].launches > 0 && blocks <= n_waves && blocks * kThreads <= (int64_t)UINT32_MAX
             ? p : single;
}

hipError_t launch_steps9(const Variant &v, const void *src, void *dst, const TileArgs &a, const MeshArgs &m,
                         const int32_t shape[3], const int32_t tgrid[3], uint32_t periodic, int steps, double omega,
                         hipStream_t s) {
  if (a.n_waves == 0) return hipSuccess;
  if (v.q != 9 || v.storage == LBM_F16_OFFSET || shape[2] != 1 || steps < 1 || steps > kMostSteps || src == dst)
    return hipErrorInvalidValue;
  Window w{shape[0], shape[1], tgrid[0], (int)periodic, steps, windows(shape[0], steps)};
  const unsigned blocks = (unsigned)((int64_t)w.wx * windows(shape[1], steps));
  auto go = [&](auto sc, auto ic, auto mc) -> hipError_t {
    constexpr int S = decltype(sc)::value;
    auto kern = k_steps9<S, decltype(ic)::value, decltype(mc)::value>;
    constexpr int lds = (8 * (int)sizeof(typename Store<S>::R) + 1) * kArea;
    if (lds > 65536) {
      const hipError_t e = hipFuncSetAttribute(reinterpret_cast<const void *>(kern),
                                               hipFuncAttributeMaxDynamicSharedMemorySize, lds);
      if (e != hipSuccess) return e;
    }
    hipLaunchKernelGGL(kern, dim3(blocks), dim3(kThreads), lds, s, src, dst, a, m.tmap, w, omega);
    return hipGetLastError();
  };
  auto by_model = [&](auto sc, auto mc) {
    return v.model == LBM_MODEL_INCOMPRESSIBLE ? go(sc, std::true_type{}, mc) : go(sc, std::false_type{}, mc);
  };
  auto by_collision = [&](auto sc) {
    return v.collision == LBM_COLLISION_MRT ? by_model(sc, std::true_type{}) : by_model(sc, std::false_type{});
  };
  return v.storage == LBM_F64 ? by_collision(std::integral_constant<int, LBM_F64>{})
                              : by_collision(std::integral_constant<int, LBM_F32_OFFSET>{});
}

}  // namespace lbm
