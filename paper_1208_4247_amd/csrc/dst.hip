// dst.hip -- exact solve of the discrete Poisson problem (the 5-/7-point
// scheme with zero Dirichlet data, Sec. 2.2) by the discrete sine transform
// (DST-I), the fast direct method the paper compares full multigrid with
// (Sec. 5.4, Tables 12-15).  The sine modes prod_i sin(k_i pi x_i) are the
// eigenvectors of A with eigenvalues sum_i (4/h^2) sin^2(k_i pi h / 2), so
//   u = S^-1 diag(lambda)^-1 S f,   S = DST-I along every axis.
//
// One DST-I of length m along the contiguous axis of an array: the odd
// extension (0, x_1 .. x_m, 0, -x_m .. -x_1) of a line, length N = 2(m+1),
// is real and odd, so its DFT is purely imaginary with coefficient k equal
// to -2i sum_j x_j sin(pi j k/(m+1)).  Two lines a, b therefore share one
// complex FFT of z = ext_a + i ext_b: Z_k = -2i S_a(k) + 2 S_b(k), so
// S_a(k) = -Im Z_k / 2 and S_b(k) = Re Z_k / 2, with no post-processing.
//   pack    the odd extensions of f's lines as complex lines (pairing below)
//   FFT     a batched complex FFT of length N (rocFFT, used as a library)
//   unpack  S(k) for every line, written with the transformed axis moved to
//           the slowest position (an LDS tile transpose)
// Pairing: a pass's m^(d-1) lines are numbered l = a o + s with o = m in 3D
// (a, s the two untransformed axes, a the slower) and o = 1 in 2D (s = 0);
// lines a and a+1 (a even) with the same s form complex line (a/2) o + s,
// line a in the real part (an odd count of a leaves the last imaginary parts
// zero).  The unpack moves mode k to the slow axis, so modes k and k+1 of a
// line land in one complex line of the next pass: every pack and unpack
// thread reads and writes whole complex values.
// so d passes visit every axis and return the array to its own axis order.
// Only f is packed by a kernel of its own: every unpack but the last writes
// its result directly as the next pass's complex lines, into the buffer the
// FFT has just consumed.
// The last forward pass divides by the eigenvalues and applies the inverse's
// scale (2/(m+1))^d (DST-I is its own inverse up to (m+1)/2 per axis); d
// more passes invert the transform.  FP64 throughout.
//
// That is the general path (a line's FFT longer than the LDS holds, 2D beyond
// 4095^2, and the one-node grids).  Everything else takes the axis kernel
// (k_dst_axis): one launch transforms every line along one axis, with the
// whole FFT of a pair of lines in LDS, in place in u.  Nothing is packed,
// extended or transposed in memory, so a pass moves 16 B per point instead of
// about 64, and the last axis runs forward transform, eigenvalue division and
// inverse in one launch: 2 d - 1 passes in all.
#include <rocfft/rocfft.h>

#include <algorithm>
#include <cmath>
#include <cstring>
#include <new>
#include <vector>

#include "../../include/gmg.h"
#include "gmg_internal.h"

namespace gmg {

// Pack f: thread t of complex line c = (a/2) o + s reads element t of lines
// a o + s and (a+1) o + s (zero past the last a) and writes both halves of
// the odd extension; the thread of t = m writes the two zeros.  blockIdx.x
// covers t, blockIdx.y strides over the complex lines.
__global__ void __launch_bounds__(256) k_dst_pack(const double *__restrict__ src,
                                                  double2 *__restrict__ z, int m, int o) {
  const int t = blockIdx.x * 256 + threadIdx.x;
  if (t > m) return;
  const size_t N = 2 * (size_t)(m + 1);
  const size_t ncl = (size_t)((m + 1) / 2) * o;
  for (size_t c = blockIdx.y; c < ncl; c += gridDim.y) {
    double2 *zl = z + c * N;
    if (t == m) {
      zl[0] = make_double2(0.0, 0.0);
      zl[m + 1] = make_double2(0.0, 0.0);
      continue;
    }
    const int a = 2 * (int)(c / o), sx = (int)(c % o);
    const double va = src[((size_t)a * o + sx) * m + t];
    const double vb = a + 1 < m ? src[((size_t)(a + 1) * o + sx) * m + t] : 0.0;
    zl[t + 1] = make_double2(va, vb);
    zl[N - 1 - t] = make_double2(-va, -vb);
  }
}

// 1/lambda times `scale` for mode k along the axis just transformed; the
// line's index holds the (0-based) modes of the other axes
template <int DIM>
__device__ __forceinline__ double dst_eig(int m, size_t line, int k, double scale,
                                          double inv_h2) {
  const double t = M_PI / (2.0 * (m + 1));
  auto s2 = [&](long q) {
    const double sv = sin(t * (double)q);
    return sv * sv;
  };
  double lam = s2(k);
  if (DIM == 2) {
    lam += s2((long)line + 1);
  } else {
    lam += s2((long)(line / m) + 1) + s2((long)(line % m) + 1);
  }
  return scale / (4.0 * inv_h2 * lam);
}

// Unpack with transpose.  A workgroup takes 32 complex lines (3D: a pair
// (a, a+1) = 2 blockIdx.z + {0, 1} and s = 32 blockIdx.y + r; 2D: a = 64
// blockIdx.y + 2 r + {0, 1}) times 32 modes k = 1 + 32 blockIdx.x + kk,
// reads them as whole complex values into LDS, then writes modes k, k+1 (k
// odd) of each line l = a o + s as one complex value of the next pass: line
// (k-1) o + l / m, element l % m, i.e. complex line ((k-1)/2) o + l / m
// (EXT); or, for the last pass, into out[(k-1) m^(d-1) + l].  eig != 0 (the
// last forward pass): divide by the eigenvalue and multiply by `scale`.
template <int DIM, bool EXT>
__global__ void __launch_bounds__(256) k_dst_unpack(const double2 *__restrict__ Z,
                                                    void *__restrict__ out, int m, int eig,
                                                    double scale, double inv_h2) {
  __shared__ double tile[2][32][33];  // [line of the pair][row r][mode kk]
  const int o = DIM == 3 ? m : 1;
  const size_t lines = (size_t)m * o;
  const size_t N = 2 * (size_t)(m + 1);
  const size_t ncl = (size_t)((m + 1) / 2) * o;
  const int k0 = 1 + blockIdx.x * 32;
  const int tx = threadIdx.x & 31, ty = threadIdx.x >> 5;  // 32 x 8
  for (int r = ty; r < 32; r += 8) {
    size_t c;
    bool ok;
    if (DIM == 3) {
      const int sx = blockIdx.y * 32 + r;
      c = (size_t)blockIdx.z * o + sx;
      ok = sx < o;
    } else {
      c = (size_t)blockIdx.y * 32 + r;
      ok = c < ncl;
    }
    const int k = k0 + tx;
    const double2 v = (ok && k <= m) ? Z[c * N + k] : make_double2(0.0, 0.0);
    tile[0][r][tx] = -0.5 * v.y;  // line a: real part of its extension
    tile[1][r][tx] = 0.5 * v.x;   // line a+1: imaginary part
  }
  __syncthreads();
  const int r = tx;
  for (int j = ty; j < 32; j += 8) {
    const int ai = j & 1, kk = 2 * (j >> 1);
    const int a = DIM == 3 ? 2 * (int)blockIdx.z + ai : (int)blockIdx.y * 64 + 2 * r + ai;
    const int sx = DIM == 3 ? (int)blockIdx.y * 32 + r : 0;
    const int k = k0 + kk;
    if (a >= m || sx >= o || k > m) continue;
    const size_t line = (size_t)a * o + sx;
    const bool has1 = k + 1 <= m;
    double v0 = tile[ai][r][kk];
    double v1 = has1 ? tile[ai][r][kk + 1] : 0.0;
    if (eig) {
      v0 *= dst_eig<DIM>(m, line, k, scale, inv_h2);
      if (has1) v1 *= dst_eig<DIM>(m, line, k + 1, scale, inv_h2);
    }
    if (EXT) {
      // next pass: line (k-1) o + a (3D) / k-1 (2D), element s (3D) / a (2D)
      const int te = DIM == 3 ? sx : a;
      double2 *zl = (double2 *)out + ((size_t)((k - 1) >> 1) * o + (DIM == 3 ? a : 0)) * N;
      zl[te + 1] = make_double2(v0, v1);
      zl[N - 1 - te] = make_double2(-v0, -v1);
      if (te == 0) {
        zl[0] = make_double2(0.0, 0.0);
        zl[m + 1] = make_double2(0.0, 0.0);
      }
    } else {
      double *d = (double *)out;
      d[(size_t)(k - 1) * lines + line] = v0;
      if (has1) d[(size_t)k * lines + line] = v1;
    }
  }
}


// ---------------------------------------------------------------- axis kernel
// DST-I along one axis, in place in LDS.  A pair of lines is the complex
// sequence z_j = a_j + i b_j, j = 1 .. m; its odd extension of length N = 2^LOGN
// = 2(m+1) is never formed: the first stage reads element j > N/2 as -z_{N-j}.
// The FFT is Stockham's (natural order in and out) in radix-8 stages with a
// radix-2 or radix-4 one at the end when 3 does not divide LOGN; N/8 threads
// hold a pair's values in registers between stages and exchange them through
// LDS.  A pair with N <= 512 lives in one wavefront and needs no barrier.  Only
// the coefficients 1 .. m are formed by the last stage.
//
// A workgroup of T threads takes P = 8 T / N pairs: consecutive rows (ROWS,
// the contiguous axis: every load and store is a run along x), or P adjacent
// pairs of columns (x, x + 1), loaded and stored as runs of 16 P bytes of each
// row of the strided axis.  EIG: forward transform, times scale / lambda, and
// inverse transform of the same axis.
//
// Bound: memory, 16 B per point and pass (LDS moves 64 B per point, the FFT
// takes about 50 operations).  A solve against rocFFT with pack and unpack
// kernels (6 passes of about 64 B): 255^3 0.38 against 1.23 ms (66-74 us a
// pass, 3.6-4.0 TB/s, 115 us the one with both transforms), 511^3 4.6 against
// 9.3, 1023^3 42.5 against 78.8, 2D 4095^2 0.69 against 0.94 ms.
// Padding: one element in 8 within a line (stage 1 writes runs of 8 per
// thread), and lines 8 elements off a multiple of 16 (a strided tile's loads
// write P lines at a time): both conflict-free.
struct DstAxisArgs {
  const double *src;
  double *dst;        // may be src
  const double2 *tw;  // exp(-2 pi i k / N), k = 0 .. N - 1
  const double *eig;  // (4 / h^2) sin^2(k pi h / 2), k = 1 .. m
  size_t stride;      // strided: elements between neighbours along the axis
  size_t outer;       // strided: elements between consecutive outer indices
  int m;
  int pairs;          // pairs of lines: in all (ROWS), per outer index (strided)
  int rows;           // ROWS: lines in all
  int nblk, gsh;
  int dim;
  double scale;
};

// Threads of a workgroup.  LDS holds 8 pairs of N = 1024 per CU however they
// are grouped, and a workgroup of several wavefronts per pair waits at its
// barriers, so small workgroups overlap better: rows take 256 threads (or one
// pair).  Strided tiles want long runs along x: 8 pairs (128 bytes) up to N =
// 512, 4 and 2 pairs beyond (the runs of neighbouring workgroups share lines
// in one XCD's L2).  1024 threads everywhere from N = 1024 on: 511^3 5.15
// against 4.57 ms, 1023^3 49.1 against 42.5 ms, 2D 511^2 48 against 27 us.
constexpr int dst_threads(int logn, bool rows) {
  const int tp = (1 << logn) / 8;
  if (rows) return tp > 256 ? tp : 256;
  return logn >= 12 ? 1024 : logn >= 9 ? 512 : 256;
}
constexpr int dst_line(int logn) { return (1 << logn) + (1 << logn) / 8 + 8; }  // LDS elements
constexpr size_t dst_lds(int logn, bool rows) {
  return (size_t)(dst_threads(logn, rows) * 8 >> logn) * dst_line(logn) * sizeof(double2);
}

__device__ __forceinline__ double2 c_add(double2 a, double2 b) { return {a.x + b.x, a.y + b.y}; }
__device__ __forceinline__ double2 c_sub(double2 a, double2 b) { return {a.x - b.x, a.y - b.y}; }
__device__ __forceinline__ double2 c_mul(double2 a, double2 b) {
  return {fma(a.x, b.x, -(a.y * b.y)), fma(a.x, b.y, a.y * b.x)};
}
__device__ __forceinline__ double2 c_mi(double2 a) { return {a.y, -a.x}; }  // times -i

template <int R>
__device__ __forceinline__ void c_fft(double2 *v) {
  if constexpr (R == 2) {
    const double2 t = v[1];
    v[1] = c_sub(v[0], t);
    v[0] = c_add(v[0], t);
  } else if constexpr (R == 4) {
    const double2 a = c_add(v[0], v[2]), b = c_sub(v[0], v[2]);
    const double2 c = c_add(v[1], v[3]), d = c_mi(c_sub(v[1], v[3]));
    v[0] = c_add(a, c);
    v[1] = c_add(b, d);
    v[2] = c_sub(a, c);
    v[3] = c_sub(b, d);
  } else {
    double2 e[4] = {v[0], v[2], v[4], v[6]}, o[4] = {v[1], v[3], v[5], v[7]};
    c_fft<4>(e);
    c_fft<4>(o);
    const double q = 0x1.6a09e667f3bcdp-1;  // sqrt(1/2)
    o[1] = {q * (o[1].x + o[1].y), q * (o[1].y - o[1].x)};
    o[2] = c_mi(o[2]);
    o[3] = {q * (o[3].y - o[3].x), -(q * (o[3].x + o[3].y))};
#pragma unroll
    for (int k = 0; k < 4; ++k) {
      v[k] = c_add(e[k], o[k]);
      v[k + 4] = c_sub(e[k], o[k]);
    }
  }
}

template <int LOGN>
struct DstLine {
  static constexpr int N = 1 << LOGN, TP = N / 8;
  static constexpr int RL = LOGN % 3 == 0 ? 8 : LOGN % 3 == 1 ? 2 : 4;  // last stage's radix
  static __device__ __forceinline__ int pad(int i) { return i + (i >> 3); }
  // the pair's threads have done their LDS accesses
  static __device__ __forceinline__ void sync() {
    if constexpr (TP <= 64)
      asm volatile("s_waitcnt lgkmcnt(0)" ::: "memory");
    else
      __syncthreads();
  }
  // stage with radix 8 (not the last unless LOGN == 3)
  template <int NS>
  static __device__ __forceinline__ void twiddle8(double2 *v, int t, const GMG_GLOBAL double2 *tw) {
    const int b = (t & (NS - 1)) * (N / (8 * NS));
#pragma unroll
    for (int k = 1; k < 8; ++k) v[k] = c_mul(v[k], double2{tw[k * b].x, tw[k * b].y});
  }
  template <int NS>
  static __device__ __forceinline__ void stages(double2 *z, double2 *v, int t,
                                                const GMG_GLOBAL double2 *tw) {
    if constexpr (NS * 8 < N || (NS * 8 == N && RL == 8)) {
      if constexpr (NS > 1) {
        sync();
#pragma unroll
        for (int k = 0; k < 8; ++k) v[k] = z[pad(t + k * TP)];
        twiddle8<NS>(v, t, tw);
      }
      c_fft<8>(v);
      if constexpr (NS * 8 == N) return;  // last: coefficient t + k N / 8 is v[k]
      sync();
      const int d = (t / NS) * (8 * NS) + (t & (NS - 1));
#pragma unroll
      for (int k = 0; k < 8; ++k) z[pad(d + k * NS)] = v[k];
      stages<NS * 8>(z, v, t, tw);
    } else {
      // radix 2 or 4: 8 / RL butterflies b = t + h TP, coefficients b + k NS
      sync();
#pragma unroll
      for (int h = 0; h < 8 / RL; ++h) {
        const int b = t + h * TP;
        double2 *w = v + h * RL;
#pragma unroll
        for (int k = 0; k < RL; ++k) {
          w[k] = z[pad(b + k * NS)];
          if (k > 0) w[k] = c_mul(w[k], double2{tw[k * b].x, tw[k * b].y});
        }
        c_fft<RL>(w);
      }
    }
  }
  // the sine coefficients of the pair staged at z (z_0 = z_{N/2} = 0): fn(k,
  // a_k, b_k) for this thread's k in 1 .. m, twice the DST-I of each line
  template <typename F>
  static __device__ __forceinline__ void dst(double2 *z, int t, const GMG_GLOBAL double2 *tw, F fn) {
    double2 v[8];
    sync();
#pragma unroll
    for (int k = 0; k < 8; ++k) {
      const double2 x = z[pad(k < 4 ? t + k * TP : (8 - k) * TP - t)];
      v[k] = k < 4 ? x : double2{-x.x, -x.y};
    }
    stages<1>(z, v, t, tw);
    sync();
#pragma unroll
    for (int h = 0; h < 8 / RL; ++h)
#pragma unroll
      for (int k = 0; k < RL / 2; ++k) {
        const int q = t + h * TP + k * (N / RL);
        const double2 w = v[h * RL + k];
        if (q > 0) fn(q, -w.y, w.x);
      }
  }
};

template <int LOGN, bool ROWS, bool EIG>
__global__ void __launch_bounds__(dst_threads(LOGN, ROWS)) k_dst_axis(DstAxisArgs a) {
  using L = DstLine<LOGN>;
  constexpr int T = dst_threads(LOGN, ROWS), TP = L::TP, P = T / TP, LS = dst_line(LOGN);
  extern __shared__ __align__(16) unsigned char smem_raw[];
  double2 *sm = reinterpret_cast<double2 *>(smem_raw);
  const int m = a.m, tid = threadIdx.x;
  const int q = tid / TP, t = tid % TP;  // this thread's pair and place in it
  double2 *z = sm + q * LS;
  const GMG_GLOBAL double2 *tw = gbl(a.tw);
  const int j = xcd_remap(blockIdx.x, a.nblk, a.gsh);
  if (t == 0) z[0] = z[L::pad(m + 1)] = double2{0.0, 0.0};
  if constexpr (ROWS) {
    const int pr = j * P + q;
    const bool ra = 2 * pr < a.rows, rb = 2 * pr + 1 < a.rows;
    const GMG_GLOBAL double *pa = gbl(a.src) + (size_t)(2 * pr) * m, *pb = pa + m;
    for (int i = t; i < m; i += TP) {
      const double x = ra ? pa[i] : 0.0, y = rb ? pb[i] : 0.0;
      z[L::pad(i + 1)] = double2{x, y};
    }
    GMG_GLOBAL double *da = gbl(a.dst) + (size_t)(2 * pr) * m, *db = da + m;
    L::dst(z, t, tw, [&](int k, double x, double y) {
      if (ra) da[k - 1] = x;
      if (rb) db[k - 1] = y;
    });
  } else {
    const int nb = (a.pairs + P - 1) / P;  // workgroups per outer index
    const int o = j / nb, p0 = (j - o * nb) * P;
    const int lp = tid % P, x = 2 * (p0 + lp);  // loads and stores: this thread's pair
    const bool in0 = x < m, in1 = x + 1 < m;
    const size_t off = (size_t)o * a.outer + x;
    double2 *zl = sm + lp * LS;
    for (int i = tid / P; i < m; i += TP) {
      const GMG_GLOBAL double *s = gbl(a.src) + off + i * a.stride;
      double2 v{0.0, 0.0};
      if (in1)
        v = {s[0], s[1]};
      else if (in0)
        v.x = s[0];
      zl[L::pad(i + 1)] = v;
    }
    __syncthreads();
    if constexpr (EIG) {
      const GMG_GLOBAL double *e = gbl(a.eig);
      const int xa = 2 * (p0 + q);
      // (columns past the grid: any finite factor, they are zero)
      const double lo = a.dim == 3 ? e[o + 1] : 0.0;
      const double la = lo + e[min(xa + 1, m)], lb = lo + e[min(xa + 2, m)];
      L::dst(z, t, tw, [&](int k, double re, double im) {
        const double ek = e[k];
        z[L::pad(k)] = double2{re * (a.scale / (la + ek)), im * (a.scale / (lb + ek))};
      });
      if (t == 0) z[0] = z[L::pad(m + 1)] = double2{0.0, 0.0};
    }
    L::dst(z, t, tw, [&](int k, double re, double im) { z[L::pad(k)] = double2{re, im}; });
    __syncthreads();
    for (int i = tid / P; i < m; i += TP) {
      GMG_GLOBAL double *d = gbl(a.dst) + off + i * a.stride;
      const double2 v = zl[L::pad(i + 1)];
      if (in1) {
        d[0] = v.x;
        d[1] = v.y;
      } else if (in0) {
        d[0] = v.x;
      }
    }
  }
}

template <int LOGN, bool ROWS, bool EIG>
hipError_t run_axis(DstAxisArgs a, int outers, hipStream_t s) {
  constexpr int T = dst_threads(LOGN, ROWS), P = T * 8 >> LOGN;
  auto k = k_dst_axis<LOGN, ROWS, EIG>;
  static int gsh = 0;
  if (gsh == 0) {
    hipError_t e = hipFuncSetAttribute((const void *)k, hipFuncAttributeMaxDynamicSharedMemorySize,
                                       (int)dst_lds(LOGN, ROWS));
    if (e == hipSuccess) e = resident_shift((const void *)k, T, dst_lds(LOGN, ROWS), gsh);
    if (e != hipSuccess) return e;
  }
  a.gsh = gsh;
  a.nblk = outers * ((a.pairs + P - 1) / P);
  gmg_launch(k, dim3(a.nblk), dim3(T), dst_lds(LOGN, ROWS), s, a);
  return hipGetLastError();
}

// mode 0: rows, 1: strided (the middle axis, 3D: N <= 2048), 2: strided with the
// eigenvalue division
template <int LOGN>
hipError_t run_axis_mode(int mode, const DstAxisArgs &a, int outers, hipStream_t s) {
  if (mode == 0) return run_axis<LOGN, true, false>(a, 1, s);
  if (mode == 2) return run_axis<LOGN, false, true>(a, outers, s);
  if constexpr (LOGN <= 11) return run_axis<LOGN, false, false>(a, outers, s);
  return hipErrorInvalidValue;
}

hipError_t launch_axis(int logn, int mode, const DstAxisArgs &a, int outers, hipStream_t s) {
  switch (logn) {
#define GMG_AXIS(L) case L: return run_axis_mode<L>(mode, a, outers, s);
    GMG_AXIS(3) GMG_AXIS(4) GMG_AXIS(5) GMG_AXIS(6) GMG_AXIS(7) GMG_AXIS(8)
    GMG_AXIS(9) GMG_AXIS(10) GMG_AXIS(11) GMG_AXIS(12) GMG_AXIS(13)
#undef GMG_AXIS
    default: return hipErrorInvalidValue;
  }
}

// Whether the axis kernels run (dim, m): a pair's FFT of length 2(m+1) <= 8192
// fits LDS with its padding (148 KB), and the radix-8 first stage needs 8.
bool axis_ok(int m) { return m >= 3 && m <= 4095; }

}  // namespace gmg

using namespace gmg;

struct gmg_dst {
  int dim = 3, m = 1;
  size_t lines = 1;
  hipStream_t stream = nullptr;
  double *E = nullptr;    // odd extensions, two real lines per complex line
  double2 *C = nullptr;   // their FFT coefficients
  void *work = nullptr;   // rocFFT work buffer
  size_t work_bytes = 0;
  rocfft_plan plan = nullptr;
  rocfft_execution_info info = nullptr;
  // axis kernels: twiddles and eigenvalues, uploaded by the setup into memory
  // of the plan's own (the workspace is scratch: its contents need not outlive
  // a solve; the host copy stays until the plan goes)
  bool axis = false;
  double2 *tw = nullptr;
  double *eig = nullptr;
  std::vector<double> host;
};

namespace {

#define HIPCHK_DST(x) \
  do {                \
    if ((x) != hipSuccess) return GMG_ERR_HIP; \
  } while (0)

constexpr size_t kAlignDst = 256;
size_t up(size_t x) { return (x + kAlignDst - 1) / kAlignDst * kAlignDst; }

bool rocfft_ready() {
  static bool ok = rocfft_setup() == rocfft_status_success;
  return ok;
}

struct DstSizes {
  size_t E, C;
};
size_t dst_pairs(int dim, int m) {
  // complex lines: lines a, a+1 of the same s share one
  return (size_t)((m + 1) / 2) * (dim == 3 ? (size_t)m : 1);
}

DstSizes dst_sizes(int dim, int m) {
  const size_t bytes = dst_pairs(dim, m) * 2 * (size_t)(m + 1) * sizeof(double2);
  DstSizes s;
  s.E = up(bytes);
  s.C = up(bytes);
  return s;
}

rocfft_status make_plan(int dim, int m, rocfft_plan *plan) {
  const size_t len = 2 * (size_t)(m + 1);
  return rocfft_plan_create(plan, rocfft_placement_notinplace,
                            rocfft_transform_type_complex_forward, rocfft_precision_double, 1,
                            &len, dst_pairs(dim, m), nullptr);
}

// FFT of the complex lines in E into C, then the unpack: into the next
// pass's complex lines in E (out == NULL) or, for the last pass, into out.
hipError_t dst_pass(gmg_dst *p, double *out, int eig, double scale) {
  const int m = p->m;
  void *in[1] = {p->E};
  void *o[1] = {p->C};
  if (rocfft_execute(p->plan, in, o, p->info) != rocfft_status_success) return hipErrorUnknown;
  const double h = 1.0 / double(m + 1);
  const unsigned kt = (m + 31) / 32;
  const dim3 grid = p->dim == 3 ? dim3(kt, kt, (m + 1) / 2)
                                : dim3(kt, (unsigned)((dst_pairs(2, m) + 31) / 32), 1);
  const double2 *Z = (const double2 *)p->C;
  void *dst = out ? (void *)out : (void *)p->E;
  const double ih2 = 1.0 / (h * h);
  if (p->dim == 2) {
    if (out)
      gmg_launch((k_dst_unpack<2, false>), grid, dim3(256), 0, p->stream, Z, dst, m, eig, scale,
                 ih2);
    else
      gmg_launch((k_dst_unpack<2, true>), grid, dim3(256), 0, p->stream, Z, dst, m, eig, scale,
                 ih2);
  } else {
    if (out)
      gmg_launch((k_dst_unpack<3, false>), grid, dim3(256), 0, p->stream, Z, dst, m, eig, scale,
                 ih2);
    else
      gmg_launch((k_dst_unpack<3, true>), grid, dim3(256), 0, p->stream, Z, dst, m, eig, scale,
                 ih2);
  }
  return hipGetLastError();
}

// Set-up for the axis kernels: they need no workspace (the nominal size keeps
// the two-phase call alike for every size) and keep their tables, at most
// 164 KB, in an allocation of the plan's own.
gmg_status axis_setup(int dim, int m, void *workspace, size_t *ws_bytes, hipStream_t stream,
                      gmg_dst **out) {
  const int N = 2 * (m + 1);
  const size_t ntw = 2 * (size_t)N, nd = ntw + (size_t)m + 1;
  if (!workspace) {
    *ws_bytes = kAlignDst;
    return GMG_OK;
  }
  if (!out) return GMG_ERR_INVALID_ARG;
  if (*ws_bytes < kAlignDst || ((uintptr_t)workspace) % kAlignDst) return GMG_ERR_WORKSPACE;
  gmg_dst *p = new (std::nothrow) gmg_dst();
  if (!p) return GMG_ERR_HIP;
  try {  // nothing throws across the C entry
    p->host.resize(nd);
  } catch (const std::bad_alloc &) {
    delete p;
    return GMG_ERR_HIP;
  }
  p->axis = true;
  p->dim = dim;
  p->m = m;
  p->stream = stream;
  const long double pi = 3.141592653589793238462643383279502884L;
  for (int k = 0; k < N; ++k) {
    p->host[2 * k] = (double)cosl(2 * pi * k / N);
    p->host[2 * k + 1] = (double)-sinl(2 * pi * k / N);
  }
  const long double n2 = (long double)(m + 1) * (m + 1);
  for (int k = 0; k <= m; ++k) {
    const long double sv = sinl(pi * k / (2 * (m + 1)));
    p->host[ntw + k] = (double)(4 * n2 * sv * sv);
  }
  if (hipMalloc((void **)&p->tw, nd * sizeof(double)) != hipSuccess) {
    delete p;
    return GMG_ERR_HIP;
  }
  p->eig = (double *)p->tw + ntw;
  if (hipMemcpyAsync(p->tw, p->host.data(), nd * sizeof(double), hipMemcpyHostToDevice, stream) !=
      hipSuccess) {
    (void)hipFree(p->tw);
    delete p;
    return GMG_ERR_HIP;
  }
  *out = p;
  return GMG_OK;
}

// x (f -> u), [y,] the last axis forward, divided by the eigenvalues and
// back, [y,] x, all in place in u.
gmg_status axis_solve(gmg_dst *p, double *u, const double *f) {
  const int m = p->m, dim = p->dim;
  int logn = 1;
  while ((1 << logn) < 2 * (m + 1)) ++logn;
  DstAxisArgs a{};
  a.tw = p->tw;
  a.eig = p->eig;
  a.m = m;
  a.dim = dim;
  a.dst = u;
  // every transform of a line comes out twice its DST-I; the inverse's scale
  a.scale = std::pow(2.0 / double(m + 1), dim) * std::pow(0.25, dim);
  auto rows = [&](const double *src) {
    a.src = src;
    a.rows = dim == 3 ? m * m : m;
    a.pairs = (a.rows + 1) / 2;
    return launch_axis(logn, 0, a, 1, p->stream);
  };
  // axis 1 (y) with outer z, or the last axis with outer y (2D: no outer)
  auto strided = [&](int axis, int mode) {
    a.src = u;
    a.pairs = (m + 1) / 2;
    a.stride = axis == 1 ? (size_t)m : (size_t)m * m;
    a.outer = axis == 1 ? (size_t)m * m : (size_t)m;
    return launch_axis(logn, mode, a, dim == 3 ? m : 1, p->stream);
  };
  HIPCHK_DST(rows(f));
  if (dim == 3) HIPCHK_DST(strided(1, 1));
  HIPCHK_DST(strided(dim - 1, 2));
  if (dim == 3) HIPCHK_DST(strided(1, 1));
  HIPCHK_DST(rows(u));
  return GMG_OK;
}

}  // namespace

extern "C" {

gmg_status gmg_dst_setup(int dim, int levels, void *workspace, size_t *ws_bytes, void *stream,
                         gmg_dst **out) {
  if (!ws_bytes || (dim != 2 && dim != 3) || levels < 1) return GMG_ERR_INVALID_ARG;
  if (levels > (dim == 3 ? 10 : 14)) return GMG_ERR_INVALID_ARG;
  const int m = (1 << levels) - 1;
  if (axis_ok(m)) return axis_setup(dim, m, workspace, ws_bytes, (hipStream_t)stream, out);
  if (!rocfft_ready()) return GMG_ERR_HIP;
  rocfft_plan plan = nullptr;
  if (make_plan(dim, m, &plan) != rocfft_status_success) return GMG_ERR_HIP;
  size_t wb = 0;
  if (rocfft_plan_get_work_buffer_size(plan, &wb) != rocfft_status_success) {
    rocfft_plan_destroy(plan);
    return GMG_ERR_HIP;
  }
  const DstSizes s = dst_sizes(dim, m);
  const size_t total = s.E + s.C + up(wb);
  if (!workspace) {
    rocfft_plan_destroy(plan);
    *ws_bytes = total;
    return GMG_OK;
  }
  if (!out) {
    rocfft_plan_destroy(plan);
    return GMG_ERR_INVALID_ARG;
  }
  if (*ws_bytes < total || ((uintptr_t)workspace) % kAlignDst) {
    rocfft_plan_destroy(plan);
    return GMG_ERR_WORKSPACE;
  }
  gmg_dst *p = new gmg_dst();
  p->dim = dim;
  p->m = m;
  p->lines = dim == 3 ? (size_t)m * m : (size_t)m;
  p->stream = (hipStream_t)stream;
  char *w = (char *)workspace;
  p->E = (double *)w;
  p->C = (double2 *)(w + s.E);
  p->work = wb ? (void *)(w + s.E + s.C) : nullptr;
  p->work_bytes = wb;
  p->plan = plan;
  if (rocfft_execution_info_create(&p->info) != rocfft_status_success ||
      rocfft_execution_info_set_stream(p->info, p->stream) != rocfft_status_success ||
      (wb && rocfft_execution_info_set_work_buffer(p->info, p->work, wb) !=
                 rocfft_status_success)) {
    if (p->info) rocfft_execution_info_destroy(p->info);
    rocfft_plan_destroy(plan);
    delete p;
    return GMG_ERR_HIP;
  }
  *out = p;
  return GMG_OK;
}

gmg_status gmg_dst_solve(gmg_dst *p, double *u, const double *f) {
  if (!p || !u || !f || (const double *)u == f) return GMG_ERR_INVALID_ARG;
  if (p->axis) return axis_solve(p, u, f);
  const double scale = std::pow(2.0 / double(p->m + 1), p->dim);
  const int m = p->m;
  const dim3 pgrid((m + 1 + 255) / 256, (unsigned)std::min<size_t>(dst_pairs(p->dim, m), 65535));
  gmg_launch(k_dst_pack, pgrid, dim3(256), 0, p->stream, f, (double2 *)p->E, m,
             p->dim == 3 ? m : 1);
  if (hipGetLastError() != hipSuccess) return GMG_ERR_HIP;
  // d forward passes (the last divides by lambda), d inverse passes; only the
  // last one writes u
  for (int a = 0; a < 2 * p->dim; ++a) {
    const int eig = a == p->dim - 1;
    if (dst_pass(p, a == 2 * p->dim - 1 ? u : nullptr, eig, eig ? scale : 1.0) != hipSuccess)
      return GMG_ERR_HIP;
  }
  return GMG_OK;
}

gmg_status gmg_dst_destroy(gmg_dst *p) {
  if (!p) return GMG_ERR_INVALID_ARG;
  if (p->info) rocfft_execution_info_destroy(p->info);
  if (p->plan) rocfft_plan_destroy(p->plan);
  if (p->tw) (void)hipFree(p->tw);  // waits for solves still running
  delete p;
  return GMG_OK;
}

}  // extern "C"
