// bottom.hip -- the bottom of the V-cycle in one workgroup.
//
// The paper identifies the coarse levels as the hard part of multigrid on a
// GPU: a launch per level and colour leaves almost every compute unit idle
// (Sec. 5.3, the per-level profile of Table 10).  Here every level whose grid
// fits in LDS (side <= 15 in 3D, <= 63 in 2D) is handled by ONE workgroup in
// ONE launch: the whole sub-V-cycle (Algorithm 1 restricted to those levels,
// down to the exactly solved one-node level, see the remark on the
// coarsest-level solver) runs out of LDS with workgroup barriers between the
// colours.  In batch mode the grid has one workgroup per problem.
//
// It is a chain of dependent steps (11 per level for V(2,2)), so what counts is
// the length of a step.  Every level gives thread b = (bx, by[, bz]) the 2 x 2
// [x 2] points at storage indices 2 b .. 2 b + 1, with u and f in registers for
// the whole cycle:
//  * half of a point's neighbours are the thread's own, the colour of a local
//    point is a constant, and no index is computed inside a step;
//  * LDS holds one array per local position (dx, dy[, dz]), so neighbouring
//    threads read neighbouring elements, each with a row of zeros below index
//    0; the pad points (storage index n - 1) are held at zero in registers;
//  * the point (1, 1[, 1]) of block b is the fine centre 2 b + 1 of coarse point
//    b, so a thread restricts to the coarse point of its own index, whose
//    right-hand side goes straight to the coarse owner's slot;
//  * the levels of at most 64 blocks (15^2, 7^3 and below) run in wavefront 0
//    with no barrier, while the other wavefronts wait at one.
// (The first colour or sweep of a zero start adds the zero sum of its
// neighbours, so every value is the general expression's.)
// Before, with one point per thread and step (its index arithmetic, six LDS reads
// and a barrier: 0.33 us a step), and now: red-black V(2,2) 2D 63^2 .. 1 23.8 and
// 13.0 us, 3D 15^3 .. 1 25.6 and 16.9 us; Jacobi V(2,2) 3D 25.9 and 13.6 us; full
// multigrid 2D 58.8 and 34.7 us.
#include "gmg_internal.h"

namespace gmg {

namespace {

// The threads that run a step and how a step ends.  W = false: the whole
// workgroup, ending with a barrier.  W = true: wavefront 0 alone (lane =
// threadIdx.x < 64), ending when its LDS operations have completed; the
// "memory" clobber keeps the compiler from moving LDS accesses across it.
template <bool W>
struct Team {
  static __device__ __forceinline__ void sync() {
    if (W)
      asm volatile("s_waitcnt lgkmcnt(0)" ::: "memory");
    else
      __syncthreads();
  }
};

// Level of side 2^K - 1: blocks and LDS arrays.
template <int DIM, int K>
struct BlkLv {
  static constexpr int n = 1 << K, nb = n / 2, P = nb + 1;  // P: array pitch
  static constexpr int SZ = DIM == 3 ? P * P * P : P * P;
  static constexpr int NB = DIM == 3 ? nb * nb * nb : nb * nb;  // blocks (threads)
  static constexpr int NP = 1 << DIM;
  // first U array of level K (levels packed coarsest first)
  static constexpr int off() {
    if constexpr (K == 1)
      return 0;
    else
      return BlkLv<DIM, K - 1>::off() + NP * BlkLv<DIM, K - 1>::SZ;
  }
  // U of levels 1 .. K, then the residual arrays of level K, then slack for
  // the reads one past the last block
  static constexpr int total() { return off() + NP * SZ + (NP - 1) * SZ + P * P + P + 2; }
};

struct BlkPar {
  int nu1, nu2;
  int c0;        // red-black: first colour of a post-smoothing sweep
  double omega;  // Jacobi
};

// V-cycles and full multigrid on levels K .. 1, for every thread of the
// workgroup (or of wavefront 0).
template <typename T, int DIM, int K, int WJ>
struct BlkCycle {
  static constexpr bool WAVE = BlkLv<DIM, K>::NB <= 64;  // runs in wavefront 0
  using Lv = BlkLv<DIM, K>;
  static constexpr int NP = Lv::NP, P = Lv::P, SZ = Lv::SZ, nb = Lv::nb;
  static constexpr int ST[3] = {1, P, P * P};

  static __device__ __forceinline__ void sync() { Team<WAVE>::sync(); }
  // block coordinates of this thread
  static __device__ __forceinline__ int bc(int ax) {
    return ((int)threadIdx.x >> (ax * (K - 1))) & (nb - 1);
  }
  static __device__ __forceinline__ int at() {
    return ((DIM == 3 ? (bc(2) + 1) * P : 0) + bc(1) + 1) * P + bc(0) + 1;
  }
  // local point p is a pad of the last block along some axis
  static __device__ __forceinline__ bool pad_point(int p) {
    bool r = false;
#pragma unroll
    for (int ax = 0; ax < DIM; ++ax) r = r || (((p >> ax) & 1) && bc(ax) == nb - 1);
    return r;
  }
  static __device__ __forceinline__ T nb_sum(const T *U, const T (&u)[NP], int p, int i) {
    T nb = T(0);
#pragma unroll
    for (int ax = 0; ax < DIM; ++ax) {
      const int o = p ^ (1 << ax);
      const bool hi = (p >> ax) & 1;
      const T lo_v = hi ? u[o] : U[o * SZ + i - ST[ax]];
      const T hi_v = hi ? U[o * SZ + i + ST[ax]] : u[o];
      nb = ax == 0 ? lo_v + hi_v : (nb + lo_v) + hi_v;
    }
    return nb;
  }
  // one half-sweep and its publication; ZERO: every neighbour is still zero
  // (the colour is a template argument: chosen at run time it would index u
  // dynamically, and u would live in scratch memory)
  template <int COLOUR, bool ZERO>
  static __device__ __forceinline__ void half(bool on, T *U, T (&u)[NP], const T (&f)[NP], int i,
                                              T h2) {
    if (on) {
#pragma unroll
      for (int p = 0; p < NP; ++p) {
        if ((__builtin_popcount(p) + DIM + COLOUR) & 1) continue;
        const T nb = ZERO ? T(0) : nb_sum(U, u, p, i);
        const T v = point_solve<T, DIM>(h2, f[p], nb);
        u[p] = pad_point(p) ? T(0) : v;
        U[p * SZ + i] = u[p];
      }
    }
    sync();
  }

  // one weighted-Jacobi sweep: every point from the published values, then the
  // publication
  template <bool ZERO>
  static __device__ __forceinline__ void jacobi(bool on, T *U, T (&u)[NP], const T (&f)[NP], int i,
                                                T h2, T omega) {
    T v[NP];
    if (on) {
#pragma unroll
      for (int p = 0; p < NP; ++p) {
        const T nb = ZERO ? T(0) : nb_sum(U, u, p, i);
        v[p] = (T(1) - omega) * u[p] + omega * point_solve<T, DIM>(h2, f[p], nb);
      }
    }
    sync();
    if (on) {
#pragma unroll
      for (int p = 0; p < NP; ++p) {
        u[p] = pad_point(p) ? T(0) : v[p];
        U[p * SZ + i] = u[p];
      }
    }
    sync();
  }

  // full weighting of r (own block in registers, the low sides of the blocks
  // above in R) to the coarse point of this block's index: the fine points 2 b
  // .. 2 b + 2 along each axis, x first, then y, then z
  static __device__ __forceinline__ T weigh(const T *R, const T (&r)[NP], int i) {
    // at (gx, gy, gz) in 0 .. 2 from the block's corner
    auto rv = [&](int gx, int gy, int gz) {
      const int p = (gx & 1) | ((gy & 1) << 1) | ((gz & 1) << 2);
      const int d = (gx >> 1) + (gy >> 1) * P + (gz >> 1) * P * P;
      return d ? R[p * SZ + i + d] : r[p];
    };
    auto row = [&](int gy, int gz) {
      return T(0.25) * rv(0, gy, gz) + T(0.5) * rv(1, gy, gz) + T(0.25) * rv(2, gy, gz);
    };
    auto plane = [&](int gz) {
      return T(0.25) * row(0, gz) + T(0.5) * row(1, gz) + T(0.25) * row(2, gz);
    };
    return DIM == 3 ? T(0.25) * plane(0) + T(0.5) * plane(1) + T(0.25) * plane(2) : plane(0);
  }

  // restrict r and solve the levels below (FMG: by full multigrid); their
  // solution is in U of level K - 1 afterwards
  template <bool FMG>
  static __device__ __forceinline__ void below(const BlkPar a, T *sm, T *R, const T (&r)[NP], bool on,
                                               int i) {
    if (on) {
#pragma unroll
      for (int p = 0; p < NP - 1; ++p) R[p * SZ + i] = r[p];
    }
    sync();
    T fc = T(0);
    if (on) fc = weigh(R, r, i);
    using C = BlkLv<DIM, K - 1>;
    T *Uc = sm + C::off();
    if constexpr (K == 2) {
      // one-node level: 2d u / h^2 = f, in FP64
      if (threadIdx.x == 0) {
        const double hc = 0.5;
        Uc[C::SZ - 1] = T((hc * hc * double(fc)) / double(2 * DIM));
      }
      sync();
    } else {
      // the right-hand side waits in the coarse owner's own slots of U
      if (on) {
        int p = 0, j = 0;
#pragma unroll
        for (int ax = DIM - 1; ax >= 0; --ax) {
          p |= (bc(ax) & 1) << ax;
          j = j * C::P + (bc(ax) >> 1) + 1;
        }
        Uc[p * C::SZ + j] = fc;
      }
      sync();
      using Sub = BlkCycle<T, DIM, K - 1, WJ>;
      if (!Sub::WAVE || threadIdx.x < 64) {
        T uc[NP], fcb[NP];
        const int j = Sub::at();
#pragma unroll
        for (int p = 0; p < NP; ++p)
          fcb[p] = (int)threadIdx.x < C::NB ? Uc[p * C::SZ + j] : T(0);
        if constexpr (FMG)
          Sub::fmg(a, sm, R, uc, fcb);
        else
          Sub::template cycle<true>(a, sm, R, uc, fcb);
      }
      if constexpr (Sub::WAVE && !WAVE) __syncthreads();
    }
  }

  // u += P u_{K-1} and its publication (coarse points b - 1 and b along each axis)
  static __device__ __forceinline__ void above(T *sm, T *U, T (&u)[NP], bool on, int i) {
    using C = BlkLv<DIM, K - 1>;
    const T *Uc = sm + C::off();
    if (on) {
      T v[2][2][2];
#pragma unroll
      for (int dz = 0; dz < (DIM == 3 ? 2 : 1); ++dz)
#pragma unroll
        for (int dy = 0; dy < 2; ++dy)
#pragma unroll
          for (int dx = 0; dx < 2; ++dx) {
            const int cx = bc(0) - 1 + dx, cy = bc(1) - 1 + dy, cz = DIM == 3 ? bc(2) - 1 + dz : 0;
            const int p = (cx & 1) | ((cy & 1) << 1) | (DIM == 3 ? (cz & 1) << 2 : 0);
            const int j = ((DIM == 3 ? ((cz >> 1) + 1) * C::P : 0) + (cy >> 1) + 1) * C::P +
                          (cx >> 1) + 1;
            v[dz][dy][dx] = Uc[p * C::SZ + j];
          }
#pragma unroll
      for (int p = 0; p < NP; ++p) {
        auto xs = [&](int dz, int dy) {
          return (p & 1) ? v[dz][dy][1] : T(0.5) * (v[dz][dy][0] + v[dz][dy][1]);
        };
        auto ys = [&](int dz) { return (p & 2) ? xs(dz, 1) : T(0.5) * (xs(dz, 0) + xs(dz, 1)); };
        T e;
        if (DIM == 3)
          e = (p & 4) ? ys(1) : T(0.5) * (ys(0) + ys(1));
        else
          e = ys(0);
        u[p] = pad_point(p) ? T(0) : u[p] + e;
        U[p * SZ + i] = u[p];
      }
    }
    sync();
  }

  // V-cycle on levels K .. 1 from u (ZERO: u is zero, neither set nor
  // published; else published)
  template <bool ZERO>
  static __device__ __forceinline__ void cycle(const BlkPar a, T *sm, T *R, T (&u)[NP],
                                               const T (&f)[NP]) {
    // (threads beyond the level's blocks take part in the barriers only)
    const bool on = (int)threadIdx.x < Lv::NB;
    T *U = sm + Lv::off();
    const int i = at();
    const T h = ldexp(T(1), -K), h2 = h * h, inv_h2 = T(Lv::n) * T(Lv::n);
    const T omega = T(a.omega);
    if (ZERO) {
#pragma unroll
      for (int p = 0; p < NP; ++p) u[p] = T(0);
    }
    for (int s = 0; s < a.nu1; ++s) {
      if constexpr (WJ) {
        if (ZERO && s == 0)
          jacobi<true>(on, U, u, f, i, h2, omega);
        else
          jacobi<false>(on, U, u, f, i, h2, omega);
      } else {
        if (ZERO && s == 0)
          half<0, true>(on, U, u, f, i, h2);
        else
          half<0, false>(on, U, u, f, i, h2);
        half<1, false>(on, U, u, f, i, h2);
      }
    }
    if (ZERO && a.nu1 == 0) {
      if (on) {
#pragma unroll
        for (int p = 0; p < NP; ++p) U[p * SZ + i] = T(0);
      }
      sync();
    }
    T r[NP];
    if (on) {
#pragma unroll
      for (int p = 0; p < NP; ++p)
        r[p] = f[p] - (T(2 * DIM) * u[p] - nb_sum(U, u, p, i)) * inv_h2;
    }
    below<false>(a, sm, R, r, on, i);
    above(sm, U, u, on, i);
    if constexpr (WJ) {
      for (int s = 0; s < a.nu2; ++s) jacobi<false>(on, U, u, f, i, h2, omega);
    } else {
      if (a.c0 == 0) half<0, false>(on && a.nu2 > 0, U, u, f, i, h2);
      for (int s = 0; s < a.nu2; ++s) {
        half<1, false>(on, U, u, f, i, h2);
        if (a.c0 == 1 || s + 1 < a.nu2) half<0, false>(on, U, u, f, i, h2);
      }
    }
  }

  // Algorithm 2 on levels K .. 1: f to the level below (full weighting, the
  // residual of the zero iterate), its solution interpolated, one V-cycle
  static __device__ __forceinline__ void fmg(const BlkPar a, T *sm, T *R, T (&u)[NP],
                                             const T (&f)[NP]) {
    const bool on = (int)threadIdx.x < Lv::NB;
    const int i = at();
#pragma unroll
    for (int p = 0; p < NP; ++p) u[p] = T(0);
    below<true>(a, sm, R, f, on, i);
    above(sm, sm + Lv::off(), u, on, i);
    cycle<false>(a, sm, R, u, f);
  }
};

template <typename T, int DIM, int K, int WJ, bool FMG>
__device__ __forceinline__ void blk_bottom(const GMG_GLOBAL T *fin, GMG_GLOBAL T *uout,
                                           const int *active, const BlkPar a, T *sm) {
  using Lv = BlkLv<DIM, K>;
  using Cy = BlkCycle<T, DIM, K, WJ>;
  constexpr int m = Lv::n - 1;
  const bool on = (int)threadIdx.x < Lv::NB;
  auto point = [&](int p, int &g) {  // global index of local point p; false: none
    const int x = 2 * Cy::bc(0) + (p & 1), y = 2 * Cy::bc(1) + ((p >> 1) & 1);
    const int z = DIM == 3 ? 2 * Cy::bc(2) + (p >> 2) : 0;
    g = (z * m + y) * m + x;
    return on && x < m && y < m && z < m;
  };
  T f[Lv::NP], u[Lv::NP];
#pragma unroll
  for (int p = 0; p < Lv::NP; ++p) {
    int g;
    f[p] = point(p, g) ? fin[g] : T(0);
  }
  // (the right-hand side is on its way before the flag is read)
  if (active && *gbl(active) == 0) return;
  // zero rows below index 0 of every array, and the one-node level
  for (int i = threadIdx.x; i < Lv::off() + Lv::NP * Lv::SZ; i += blockDim.x) sm[i] = T(0);
  __syncthreads();
  if (Cy::WAVE && threadIdx.x >= 64) return;  // (no barrier after this)
  T *const R = sm + Lv::off() + Lv::NP * Lv::SZ;
  if constexpr (FMG)
    Cy::fmg(a, sm, R, u, f);
  else
    Cy::template cycle<true>(a, sm, R, u, f);
#pragma unroll
  for (int p = 0; p < Lv::NP; ++p) {
    int g;
    if (point(p, g)) uout[g] = u[p];
  }
}

constexpr int blk_threads(int dim, int L) {
  return dim == 3 ? (L >= 4 ? 512 : 64) : (L >= 6 ? 1024 : L == 5 ? 256 : 64);
}
template <int DIM>
size_t blk_lds(int L, size_t elem) {
  int n = 1;
  switch (L) {
    case 2: n = BlkLv<DIM, 2>::total(); break;
    case 3: n = BlkLv<DIM, 3>::total(); break;
    case 4: n = BlkLv<DIM, 4>::total(); break;
    case 5: n = BlkLv<DIM, 5>::total(); break;
    case 6: n = BlkLv<DIM, 6>::total(); break;
  }
  return n * elem;
}

}  // namespace

// One workgroup per problem (batch: one table entry each, of at most the
// launch's level count).
template <typename T, int DIM, int WJ, bool FMG>
__global__ void __launch_bounds__(DIM == 3 ? 512 : 1024) k_bottom(BottomArgs<T> arg,
                                                                  const BottomArgs<T> *tbl) {
  const int *active = arg.active;
  const T *fp = arg.f;
  T *up = arg.u;
  int L = arg.L;
  BlkPar par{arg.nu1, arg.nu2, arg.post_forward ? 0 : 1, arg.omega};
  if (tbl) {
    const BottomArgs<T> *e = tbl + blockIdx.x;
    active = e->active;
    fp = e->f;
    up = e->u;
    L = e->L;
    par = BlkPar{e->nu1, e->nu2, e->post_forward ? 0 : 1, e->omega};
  }
  const GMG_GLOBAL T *fin = gbl(fp);
  GMG_GLOBAL T *uout = gbl(up);
  extern __shared__ __align__(16) unsigned char smem_raw[];
  T *sm = reinterpret_cast<T *>(smem_raw);
  switch (L) {
    case 1:
      if (threadIdx.x == 0 && !(active && *gbl(active) == 0)) {  // 2d u / h^2 = f, h = 1/2, FP64
        const double h = 0.5;
        uout[0] = T((h * h * double(fin[0])) / double(2 * DIM));
      }
      break;
    case 2: blk_bottom<T, DIM, 2, WJ, FMG>(fin, uout, active, par, sm); break;
    case 3: blk_bottom<T, DIM, 3, WJ, FMG>(fin, uout, active, par, sm); break;
    case 4: blk_bottom<T, DIM, 4, WJ, FMG>(fin, uout, active, par, sm); break;
    case 5:
      if constexpr (DIM == 2) blk_bottom<T, DIM, 5, WJ, FMG>(fin, uout, active, par, sm);
      break;
    case 6:
      if constexpr (DIM == 2) blk_bottom<T, DIM, 6, WJ, FMG>(fin, uout, active, par, sm);
      break;
  }
}

template <typename T, int DIM, int WJ, bool FMG>
hipError_t run_bottom(int nproblems, BottomArgs<T> a, const BottomArgs<T> *tbl, hipStream_t s) {
  auto k = k_bottom<T, DIM, WJ, FMG>;
  static bool attr = false;
  if (!attr) {
    hipError_t e = hipFuncSetAttribute((const void *)k, hipFuncAttributeMaxDynamicSharedMemorySize,
                                       (int)blk_lds<DIM>(DIM == 3 ? 4 : 6, sizeof(T)));
    if (e != hipSuccess) return e;
    attr = true;
  }
  gmg_launch(k, dim3(nproblems), dim3(blk_threads(DIM, a.L)), blk_lds<DIM>(a.L, sizeof(T)), s, a,
             tbl);
  return hipGetLastError();
}

template <typename T, int DIM>
hipError_t run_bottom_dim(int nproblems, BottomArgs<T> a, const BottomArgs<T> *tbl, hipStream_t s) {
  if (a.fmg) {  // full multigrid runs FP64 plans only
    if constexpr (sizeof(T) == 8)
      return a.smoother ? run_bottom<T, DIM, 1, true>(nproblems, a, tbl, s)
                        : run_bottom<T, DIM, 0, true>(nproblems, a, tbl, s);
    else
      return hipErrorInvalidValue;
  }
  return a.smoother ? run_bottom<T, DIM, 1, false>(nproblems, a, tbl, s)
                    : run_bottom<T, DIM, 0, false>(nproblems, a, tbl, s);
}

template <typename T>
hipError_t launch_bottom(int nproblems, BottomArgs<T> a, const BottomArgs<T> *tbl, hipStream_t s) {
  if (a.L < 1 || a.L > bottom_max_levels(a.dim)) return hipErrorInvalidValue;
  return a.dim == 3 ? run_bottom_dim<T, 3>(nproblems, a, tbl, s)
                    : run_bottom_dim<T, 2>(nproblems, a, tbl, s);
}

template hipError_t launch_bottom<double>(int, BottomArgs<double>, const BottomArgs<double> *,
                                          hipStream_t);
template hipError_t launch_bottom<float>(int, BottomArgs<float>, const BottomArgs<float> *,
                                         hipStream_t);

// ------------------------------------------------------------------------
// The bottom of the paper's own cycle (multicolour Gauss-Seidel, linear
// finite-element transfers; variant.hip holds the kernels of the larger levels):
// levels of side <= 15 (3D), <= 63 (2D) in one workgroup.  One launch per half
// sweep and transfer cost 4 us each whatever the level, 27 us a level of V(1,1)
// in 3D; a colour step here is one LDS round trip of a point per thread.  3D
// 15^3 .. 1 V(1,1): 81 us by level, 15 us so (means over a solve).
//
// Node indices run 0 .. n, zero at both ends; thread b owns the nodes 2 b + o,
// o in {0, 1}^d (one point per colour), with their right-hand sides in
// registers, and restricts to and interpolates from the coarse node b.  All
// sums are in the order of the per-level kernels: the same bits.
// ------------------------------------------------------------------------
namespace {

struct VarPar {
  int nu1, nu2, backward, relax;
};

template <int DIM, int K>
struct VarCycle {
  static constexpr int n = 1 << K, nb = n / 2, P = n + 1, PP = DIM == 3 ? P * P : 0;
  static constexpr int SZ = DIM == 3 ? P * P * P : P * P;
  static constexpr int NB = DIM == 3 ? nb * nb * nb : nb * nb;
  static constexpr int NP = 1 << DIM;
  static constexpr bool WAVE = NB <= 64;
  static constexpr int PC = nb + 1, PPC = DIM == 3 ? PC * PC : 0;  // coarse pitches
  // LDS: U of levels 1 .. K (coarsest first), then the residual, then the
  // coarse right-hand side (both reused by every level)
  static constexpr int off() {
    if constexpr (K == 1) return 0;
    else return VarCycle<DIM, K - 1>::off() + VarCycle<DIM, K - 1>::SZ;
  }
  static constexpr int total() { return off() + 2 * SZ + VarCycle<DIM, K - 1>::SZ; }

  static __device__ __forceinline__ int bc(int d) {
    return ((int)threadIdx.x / (d == 0 ? 1 : d == 1 ? nb : nb * nb)) % nb;
  }
  static __device__ __forceinline__ int node(int p) {  // LDS index of local point p
    return (2 * (DIM == 3 ? bc(2) : 0) + (p >> 2)) * PP + (2 * bc(1) + ((p >> 1) & 1)) * P +
           2 * bc(0) + (p & 1);
  }
  static __device__ __forceinline__ int coarse(int ox, int oy, int oz) {  // coarse node b + o
    return (DIM == 3 ? bc(2) + oz : 0) * PPC + (bc(1) + oy) * PC + bc(0) + ox;
  }
  // bit p: local point p is an interior node
  static __device__ __forceinline__ int interior() {
    int v = 0;
    if ((int)threadIdx.x >= NB) return 0;
#pragma unroll
    for (int p = 0; p < NP; ++p)
      if ((bc(0) > 0 || (p & 1)) && (bc(1) > 0 || (p & 2)) && (DIM == 2 || bc(2) > 0 || (p & 4)))
        v |= 1 << p;
    return v;
  }

  template <bool BW>
  static __device__ __forceinline__ void sweep(double *U, const double *f, int in) {
    constexpr double h = 1.0 / n, h2 = h * h, diag = 2.0 * DIM;
#pragma unroll
    for (int s = 0; s < NP; ++s) {
      const int c = BW ? NP - 1 - s : s;  // colour (i&1) + 2 (j&1) + 4 (k&1) = local point
      if (in >> c & 1) {
        const int q = node(c);
        double r = h2 * f[c];
        if (DIM == 3) r = r + (U[q - PP] + U[q + PP]);
        U[q] = (r + ((U[q - 1] + U[q + 1]) + (U[q - P] + U[q + P]))) / diag;
      }
      Team<WAVE>::sync();
    }
  }
  static __device__ __forceinline__ void smooth(double *U, const double *f, int in, int nsweeps,
                                                int backward) {
    for (int k = 0; k < nsweeps; ++k) {
      if (backward)
        sweep<true>(U, f, in);
      else
        sweep<false>(U, f, in);
    }
  }

  // V-cycle on this level's U (start value in LDS); f: this thread's
  // right-hand sides; sm, res, fcs: see the LDS map.  Ends synchronised.
  static __device__ __forceinline__ void cycle(const VarPar a, double *sm, double *res,
                                               double *fcs, const double *f) {
    constexpr double inv_h2 = double(n) * n, diag = 2.0 * DIM;
    double *const U = sm + off();
    const int in = interior();
    smooth(U, f, in, a.nu1, 0);
#pragma unroll
    for (int p = 0; p < NP; ++p)
      if (in >> p & 1) {
        const int q = node(p);
        double nbs = U[q - 1] + U[q + 1] + U[q - P] + U[q + P];
        if (DIM == 3) nbs = nbs + U[q - PP] + U[q + PP];
        res[q] = f[p] - (diag * U[q] - nbs) * inv_h2;
      }
    Team<WAVE>::sync();
    if (in & 1) {  // coarse node b is an interior node
      const double *r = res + node(0);
      const double mid = 2.0 * r[0] + (r[1] + r[-1]) + (r[P] + r[-P]) + (r[P + 1] + r[-P - 1]);
      double s;
      if (DIM == 3) {
        const double *lo = r - PP, *hi = r + PP;
        s = lo[0] + lo[-1] + lo[-P] + lo[-P - 1];
        s = s + mid;
        s = (s + (hi[0] + hi[1] + hi[P] + hi[P + 1])) * 0.0625;
      } else {
        s = mid * 0.125;
      }
      fcs[coarse(0, 0, 0)] = s;
    }
    Team<WAVE>::sync();
    if constexpr (K == 2) {
      if (threadIdx.x == 0) {  // one node, h = 1/2; a Gauss-Seidel sweep from zero is exact
        const int one = DIM == 3 ? 13 : 4;
        sm[one] = a.relax && a.nu1 == 0 ? 0.0 : (0.25 * fcs[one]) / diag;
      }
      Team<WAVE>::sync();
    } else {
      using Cc = VarCycle<DIM, K - 1>;
      if (!Cc::WAVE || threadIdx.x < 64) {
        double fc[NP];
        const int inc = Cc::interior();
#pragma unroll
        for (int p = 0; p < NP; ++p) fc[p] = inc >> p & 1 ? fcs[Cc::node(p)] : 0.0;
        Team<Cc::WAVE>::sync();
        Cc::cycle(a, sm, res, fcs, fc);
      }
      if (!WAVE) __syncthreads();
    }
    const double *const E = sm + VarCycle<DIM, K - 1>::off();
    if ((int)threadIdx.x < NB) {
      const double c0 = E[coarse(0, 0, 0)];
#pragma unroll
      for (int p = 0; p < NP; ++p)
        if (in >> p & 1)
          U[node(p)] += p ? 0.5 * (c0 + E[coarse(p & 1, (p >> 1) & 1, p >> 2)]) : c0;
    }
    Team<WAVE>::sync();
    smooth(U, f, in, a.nu2, a.backward);
  }

  static __device__ __forceinline__ void run(const double *uin, const double *fin, double *uout,
                                             const int *active, const VarPar a, double *sm) {
    constexpr int m = n - 1;
    const int in = interior();
    auto global = [&](int p) {  // storage index of local point p
      const int x = 2 * bc(0) + (p & 1) - 1, y = 2 * bc(1) + ((p >> 1) & 1) - 1;
      const int z = DIM == 3 ? 2 * bc(2) + (p >> 2) - 1 : 0;
      return (z * m + y) * m + x;
    };
    double f[NP], u0[NP];
#pragma unroll
    for (int p = 0; p < NP; ++p) {
      f[p] = in >> p & 1 ? gbl(fin)[global(p)] : 0.0;
      u0[p] = uin && (in >> p & 1) ? gbl(uin)[global(p)] : 0.0;
    }
    if (active && *gbl(active) == 0) return;
    for (int i = threadIdx.x; i < total(); i += blockDim.x) sm[i] = 0.0;
    __syncthreads();
    if (WAVE && threadIdx.x >= 64) return;  // (no barrier after this)
    double *const U = sm + off();
#pragma unroll
    for (int p = 0; p < NP; ++p)
      if (in >> p & 1) U[node(p)] = u0[p];
    Team<WAVE>::sync();
    cycle(a, sm, U + SZ, U + 2 * SZ, f);
#pragma unroll
    for (int p = 0; p < NP; ++p)
      if (in >> p & 1) gbl(uout)[global(p)] = U[node(p)];
  }
};

}  // namespace

template <int DIM, int K>
__global__ void __launch_bounds__(blk_threads(DIM, K)) k_var_bottom(const double *uin,
                                                                    const double *f, double *uout,
                                                                    const int *active, VarPar a) {
  extern __shared__ __align__(16) unsigned char smem_raw[];
  VarCycle<DIM, K>::run(uin, f, uout, active, a, reinterpret_cast<double *>(smem_raw));
}

template <int DIM, int K>
static hipError_t run_var_bottom(const double *uin, const double *f, double *uout,
                                 const int *active, VarPar a, hipStream_t s) {
  constexpr size_t lds = VarCycle<DIM, K>::total() * sizeof(double);
  auto k = k_var_bottom<DIM, K>;
  hipError_t e = hipFuncSetAttribute((const void *)k, hipFuncAttributeMaxDynamicSharedMemorySize,
                                     (int)lds);
  if (e != hipSuccess) return e;
  gmg_launch(k, dim3(1), dim3(blk_threads(DIM, K)), lds, s, uin, f, uout, active, a);
  return hipGetLastError();
}

hipError_t launch_var_bottom(int dim, int levels, const double *uin, const double *f, double *uout,
                             int nu1, int nu2, int backward, int relax, const int *active,
                             hipStream_t s) {
  const VarPar a{nu1, nu2, backward, relax};
  if (dim == 3) {
    switch (levels) {
      case 2: return run_var_bottom<3, 2>(uin, f, uout, active, a, s);
      case 3: return run_var_bottom<3, 3>(uin, f, uout, active, a, s);
      case 4: return run_var_bottom<3, 4>(uin, f, uout, active, a, s);
    }
  } else if (dim == 2) {
    switch (levels) {
      case 2: return run_var_bottom<2, 2>(uin, f, uout, active, a, s);
      case 3: return run_var_bottom<2, 3>(uin, f, uout, active, a, s);
      case 4: return run_var_bottom<2, 4>(uin, f, uout, active, a, s);
      case 5: return run_var_bottom<2, 5>(uin, f, uout, active, a, s);
      case 6: return run_var_bottom<2, 6>(uin, f, uout, active, a, s);
    }
  }
  return hipErrorInvalidValue;
}

}  // namespace gmg
