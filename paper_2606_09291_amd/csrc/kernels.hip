// kernels.hip -- gfx950 kernels of libmlsgd.
//
// Stencil work is HBM-bound (a few flop per byte), so the kernels are built
// for coalesced z-fastest access, LDS reuse of the (y, z) neighbours, and no
// stored coefficient: the diffusion coefficient a = exp(log a) of every
// sample is regenerated from its KL coefficients inside each sweep (Sec. 5
// model problem).  MFMA does not apply to this work.
//
// Layout: a "row" is one problem (one sample on one grid); a batch of rows of
// one grid size is [rows][n^3], z fastest, boundary entries held at zero.
#include "internal.h"

#include <hip/hip_runtime.h>

#include <algorithm>
#include <cmath>
#include <cstdio>
#include <cstdlib>
#include <type_traits>

namespace mlsgd {

// ---------------------------------------------------------------------------
// helpers
// ---------------------------------------------------------------------------
__device__ __forceinline__ double dexp(double x) { return exp(x); }
__device__ __forceinline__ float dexp(float x) { return __expf(x); }

// Reciprocal: hardware estimate refined by two Newton steps (FP64) -- within
// one ulp for the positive, O(1) arguments it sees here.
__device__ __forceinline__ double drcp(double d) {
  double r = __builtin_amdgcn_rcp(d);
  double e = __builtin_fma(-d, r, 1.0);
  r = __builtin_fma(r, e, r);
  e = __builtin_fma(-d, r, 1.0);
  r = __builtin_fma(r, e, r);
  return r;
}
__device__ __forceinline__ float drcp(float d) { return __builtin_amdgcn_rcpf(d); }

// bfloat16 storage: round to nearest even from FP32, widen by a shift.
__device__ __forceinline__ uint16_t to_bf16(float f) {
  const uint32_t u = __float_as_uint(f);
  return (uint16_t)((u + 0x7FFFu + ((u >> 16) & 1u)) >> 16);
}
__device__ __forceinline__ float from_bf16(uint16_t h) { return __uint_as_float((uint32_t)h << 16); }

// Harmonic face coefficient from the reciprocal vertex coefficients
// b = 1/a:  2 a_v a_w / (a_v + a_w) = 2 / (b_v + b_w).
template <typename T>
__device__ __forceinline__ T face(T bv, T bw) {
  return T(2) * drcp(bv + bw);
}

// Reciprocal and face of the fused smoothing passes: in FP64 one Newton step
// from the hardware estimate instead of two (within a few ulp of drcp).  The
// pre- and post-smoothing passes of a grid both use them, so the cycle stays
// symmetric: multigrid for the operator with these faces, a fixed SPD
// operator within a few ulp of A, while the Krylov matvec applies A itself.
__device__ __forceinline__ double srcp(double d) {
  const double r = __builtin_amdgcn_rcp(d);
  const double e = __builtin_fma(-d, r, 1.0);
  return __builtin_fma(r, e, r);
}
__device__ __forceinline__ float srcp(float d) { return __builtin_amdgcn_rcpf(d); }
template <typename T>
__device__ __forceinline__ T sface(T bv, T bw) {
  return T(2) * srcp(bv + bw);
}

// Workgroups are dealt round-robin to the 8 XCDs; renumber them so that each
// XCD (own L2) receives a contiguous range of logical tiles, which then share
// halo rows in that L2.
__device__ __forceinline__ int xcd_swizzle(int b, int nb) {
  const int q = nb >> 3, r = nb & 7;
  const int xcd = b & 7, loc = b >> 3;
  return (xcd < r ? xcd * (q + 1) : r * (q + 1) + (xcd - r) * q) + loc;
}

// Sum of a problem's c partial slots by LP consecutive lanes (a power of two,
// at most a wave): lane `sub` adds slots sub, sub + LP, ..., eight loads in
// flight at a time, and the lanes' sums are added in a fixed butterfly, so the
// sum is deterministic and every lane of the problem holds it.
template <int LP>
__device__ __forceinline__ double slots_sum(const double* __restrict__ v, int c, int sub) {
  double sum = 0.0;
  int j = sub;
  for (; j + 7 * LP < c; j += 8 * LP) {
    double t[8];
#pragma unroll
    for (int u = 0; u < 8; ++u) t[u] = v[j + u * LP];
#pragma unroll
    for (int u = 0; u < 8; ++u) sum += t[u];
  }
  for (; j < c; j += LP) sum += v[j];
#pragma unroll
  for (int o = LP / 2; o > 0; o >>= 1) sum += __shfl_xor(sum, o, 64);
  return sum;
}

// Wave sum on the DPP path (row shifts, then row broadcasts): lane 63 holds
// the sum of all 64 lanes, in a fixed order.
template <int CTRL, int ROWS>
__device__ __forceinline__ double dpp_add(double v) {
  union {
    double d;
    int i[2];
  } a, b;
  a.d = v;
  b.i[0] = __builtin_amdgcn_update_dpp(0, a.i[0], CTRL, ROWS, 0xf, false);
  b.i[1] = __builtin_amdgcn_update_dpp(0, a.i[1], CTRL, ROWS, 0xf, false);
  return v + b.d;
}
__device__ __forceinline__ double wave_sum63(double v) {
  v = dpp_add<0x111, 0xf>(v);   // row_shr:1
  v = dpp_add<0x112, 0xf>(v);   // row_shr:2
  v = dpp_add<0x114, 0xf>(v);   // row_shr:4
  v = dpp_add<0x118, 0xf>(v);   // row_shr:8
  v = dpp_add<0x142, 0xa>(v);   // row_bcast:15 into rows 1 and 3
  v = dpp_add<0x143, 0xc>(v);   // row_bcast:31 into rows 2 and 3
  return v;
}

template <int NT>
__device__ __forceinline__ double block_sum(double v, double* sred, int tid) {
#pragma unroll
  for (int o = 32; o > 0; o >>= 1) v += __shfl_down(v, o, 64);
  const int lane = tid & 63, w = tid >> 6;
  if (lane == 0) sred[w] = v;
  __syncthreads();
  double s = 0.0;
  if (tid == 0) {
#pragma unroll
    for (int i = 0; i < NT / 64; ++i) s += sred[i];
  }
  __syncthreads();
  return s;  // valid in thread 0
}
template <int NT>
__device__ __forceinline__ double block_sum(double v, double* sred) {
  return block_sum<NT>(v, sred, threadIdx.x);
}

static inline int cdiv(long long a, long long b) { return (int)((a + b - 1) / b); }

// Most workgroups of 256 threads in one launch: a launch holds fewer than 2^32
// threads.  Launches over several grid sizes whose workgroups add up to more are
// made in parts.
constexpr long long MAX_WG256 = (1LL << 24) - 1;

// A workgroup marches its chunk at about a memory round trip per plane, so a
// batch too small to fill the chip takes as long as one chunk.  With the batch's
// rows known, the chunk is halved (to even lengths) while that shortens the
// estimate rounds x (planes + 6): rounds of the workgroups that fit at once, the
// chunk's planes, and about six planes' worth of first loads and ring planes.  A
// gain under 15% keeps the longer chunk (each chunk repeats two ring planes),
// and grids of one 8 x 8 tile keep one chunk (k_vsmall writes their one slot).
// Measured, 32-plane chunks against the rule: one 33^3 state and adjoint solve 4.1
// -> 2.0 ms (post-smoothing 48 -> 14 us a pass), the 17^3..65^3 law workload 13.8
// -> 6.5, 300 solves of 33^3..65^3 26.7 -> 23.7; full batches keep their chunks.
// Two planes against four as the shortest chunk: one 33^3 state and adjoint solve
// 1.45 -> 1.29 ms, graph replay of a 64/16/4 estimate 1.97 -> 1.87.
static int split_chunk(const Tiling& t, int m, int rows) {
  const int threads = t.TY * t.TZ;
  const long long fit = 256LL * (threads >= 1024 ? 1 : 1024 / threads);
  auto cost = [&](int ch) {
    const long long wg = (long long)rows * t.nty * t.ntz * cdiv(m, ch);
    return ((wg + fit - 1) / fit) * (ch + 6);
  };
  int best = t.xchunk;
  // one chunk of an odd number of planes splits as the even length above it
  for (int ch = (t.nxc == 1 ? t.xchunk + (t.xchunk & 1) : t.xchunk); ch % 4 == 0;) {
    ch /= 2;
    if (100 * cost(ch) < 85 * cost(best)) best = ch;
  }
  return best;
}

// x planes of a chunk as asked for; lengths below 8 stand for the default
static int chunk_planes(int xchunk) { return xchunk >= 8 ? xchunk : 32; }

Tiling make_tiling(int n, int tile_y, int xchunk, int rows) {
  const int m = n - 2;
  Tiling t;
  if (m <= 8) {
    t.TY = 8; t.TZ = 8;
  } else if (m <= 16) {
    t.TY = 16; t.TZ = 16;
  } else if (m <= 32) {
    t.TY = 8; t.TZ = 32;
  } else {
    t.TY = (tile_y == 4 || tile_y == 16) ? tile_y : 8;
    t.TZ = 64;
  }
  const int xch = chunk_planes(xchunk);
  t.nty = cdiv(m, t.TY);
  t.ntz = cdiv(m, t.TZ);
  t.xchunk = m <= xch ? m : xch;
  t.nxc = cdiv(m, t.xchunk);
  if (rows > 0 && m > 8) {
    t.xchunk = split_chunk(t, m, rows);
    t.nxc = cdiv(m, t.xchunk);
  }
  t.tiles_per_row = t.nty * t.ntz * t.nxc;
  return t;
}

// ---------------------------------------------------------------------------
// Marching stencil kernel.
//
// A workgroup owns the (y, z) patch [y0, y0+TY) x [z0, z0+TZ) of one row and
// walks the x planes of its chunk.  Each thread keeps its own column's
// values and reciprocal coefficients at x-1, x, x+1 in registers; the
// current plane (patch plus a one-point halo in y and z) sits in LDS,
// double-buffered so one barrier per plane suffices.
//
// Coefficient: either regenerated in the sweep from the separable KL sum --
// per (y, z) column S[k1] = sum_{k2,k3} c[k1,k2,k3] cos(pi k2 y) cos(pi k3 z)
// is formed once, after which each plane costs K FMAs and one exp -- or read
// from the per-estimate cache of 1/a written by k_coef_cache (CACHED).
//
// OP_RESID : r = b - A x
// OP_MATVEC: p = z + beta p (on the fly, halo included), q = A p, <p, q>;
//            with xdef non-null also xdef += alpha p_old, the previous
//            iteration's step of the iterate (alpha still in the scalars)
// OP_GS    : one colour of a red-black Gauss-Seidel sweep in place with
//            relaxation omega (x_zero: start from x = 0; partial: <b, x>)
// OP_JAC   : one damped Jacobi step out of place, x' = x + omega D^-1 (b - A x)
//            (the steps of the Chebyshev smoother; x_zero: x = 0; partial:
//            <b, x'>); OP_JACP also adds the trilinear prolongation of the
//            coarse rows in2 to every loaded x (coarse-grid correction)
// OP_JAC2Z : the first two steps from x = 0 in one pass: every loaded x is the
//            first step's value omega1 b / D, formed from b (rhs) and the
//            stored reciprocal diagonal (in), then one Jacobi step follows
// ---------------------------------------------------------------------------
template <typename T>
__device__ __forceinline__ T prolong_val(int nc, const T* __restrict__ c, int ix, int iy, int iz) {
  const int ax = ix >> 1, bx = (ix + 1) >> 1;
  const int ay = iy >> 1, by = (iy + 1) >> 1;
  const int az = iz >> 1, bz = (iz + 1) >> 1;
  const int cp = lay_pitch(nc), co = lay_off(nc);
  auto cv = [&](int a, int b, int d) { return c[((size_t)a * nc + b) * cp + d + co]; };
  T v = cv(ax, ay, az);
  if (iz & 1) v += cv(ax, ay, bz);
  if (iy & 1) {
    v += cv(ax, by, az);
    if (iz & 1) v += cv(ax, by, bz);
  }
  if (ix & 1) {
    v += cv(bx, ay, az);
    if (iz & 1) v += cv(bx, ay, bz);
    if (iy & 1) {
      v += cv(bx, by, az);
      if (iz & 1) v += cv(bx, by, bz);
    }
  }
  const T w = ((ix & 1) ? T(0.5) : T(1)) * ((iy & 1) ? T(0.5) : T(1)) * ((iz & 1) ? T(0.5) : T(1));
  return w * v;
}

// Trilinear prolongation along one fine (y, z) column while marching in x.
// The workgroup stages each coarse plane of its tile's footprint once in an
// LDS ring (four planes); a column forms the (y, z)-bilinear value of a
// coarse plane from four LDS taps and keeps it for the three fine planes that
// use it.  A missing second tap in y or z is read at offset 0:
// 0.25 ((a + a) + (b + b)) equals 0.5 (a + b) exactly, so one formula serves
// every column parity.  Calls to at() come with ix increasing by one.
template <typename T>
struct ProlongLds {
  int lc, dyl, dzl, ja;  // slab offset of the lower taps, upper-tap offsets
  T v0, v1;              // bilinear values of coarse planes ja, ja + 1
  __device__ T bil(const T* ring, int cslab, int j) const {
    const T* p = ring + (j & 3) * cslab + lc;
    return T(0.25) * ((p[0] + p[dzl]) + (p[dyl] + p[dyl + dzl]));
  }
  __device__ void init(const T* ring, int cslab, int czn, int cy0, int cz0, int jy, int jz,
                       int ix0) {
    lc = ((jy >> 1) - cy0) * czn + ((jz >> 1) - cz0);
    dyl = (jy & 1) ? czn : 0;
    dzl = (jz & 1) ? 1 : 0;
    ja = ix0 >> 1;
    v0 = bil(ring, cslab, ja);
    v1 = bil(ring, cslab, ja + 1);
  }
  __device__ T at(const T* ring, int cslab, int ix) {
    const int j = ix >> 1;
    if (j + (ix & 1) > ja + 1) {
      v0 = v1;
      ++ja;
      v1 = bil(ring, cslab, ja + 1);
    }
    if (ix & 1) return T(0.5) * (v0 + v1);
    return j == ja ? v0 : v1;
  }
};

// A value as loaded (r, and for OP_MATVEC the old direction, for OP_JACP the
// prolonged correction, in c); it is combined one plane after the load was
// issued, so the loads of the two-plane-ahead prefetch stay in flight.
template <typename T, typename TI>
struct Ld {
  TI r;
  T c;
};

enum MarchOp { OP_RESID = 0, OP_MATVEC = 1, OP_GS = 2, OP_JAC = 3, OP_JACP = 4, OP_JAC2Z = 5 };

// LDS of one tile
template <typename T, int TY, int TZ, int OP, int CK>
struct MarchLds {
  static constexpr int PLANE = (TY + 2) * (TZ + 2);
  static constexpr int CSLAB = (TY / 2 + 2) * (TZ / 2 + 2);
  T sx[2][PLANE], sb[2][PLANE];
  double sc[CK != 0 ? 1 : KMAX * KMAX * KMAX];
  double sred[TY * TZ / 64];
  T scs[OP == OP_JACP ? 4 * CSLAB : 1];
};

// Tile `bid` of the launch over g by TY x TZ threads (tid: index among them).
template <typename T, typename TI, int TY, int TZ, int OP, int CK>
__device__ __forceinline__ void march_tile(MarchLds<T, TY, TZ, OP, CK>& lds, const GridArgs& g,
                                           int bid, int tid, const TI* in, const T* in2,
                                           const T* rhs, T* out, T* out2,
                                           const int* __restrict__ poff,
                                           double* __restrict__ partial, int color, int x_zero,
                                           int top_begin, T omega, T* __restrict__ xdef) {
  constexpr bool CACHED = CK != 0;   // 0: regenerate, 1: cache of type T, 2: bfloat16 cache
  constexpr int NT = TY * TZ;
  constexpr int PZ = TZ + 2;
  auto& sx = lds.sx;
  auto& sb = lds.sb;
  auto& sc = lds.sc;
  auto& scs = lds.scs;

  const int n = g.n;
  const int LP = lay_pitch(n), LO = lay_off(n);
  const int tpr = g.t.tiles_per_row;
  const int row = bid / tpr;
  const int tile = bid - row * tpr;
  int tt = tile;
  const int ty = tt % g.t.nty;
  tt /= g.t.nty;
  const int tz = tt % g.t.ntz;
  const int xc = tt / g.t.ntz;
  const int prob = g.row0 + row;
  if (g.scal && !g.scal[prob].active) return;  // uniform per workgroup

  const int K = g.K;
  if (!CACHED) {
    const int K3 = K * K * K;
    for (int j = tid; j < K3; j += NT) sc[j] = g.coef[(size_t)prob * K3 + j];
    __syncthreads();
  }

  const size_t base = (size_t)row * (size_t)g.stride;
  const T* __restrict__ cache = (const T*)g.cache + (size_t)prob * (size_t)g.stride;
  const uint16_t* __restrict__ cache16 = (const uint16_t*)g.cache + (size_t)prob * (size_t)g.stride;
  const double* __restrict__ cosT = g.cosT;
  const int ly = tid / TZ, lz = tid - (tid / TZ) * TZ;
  const int y0 = 1 + ty * TY, z0 = 1 + tz * TZ;
  const int iy = y0 + ly, iz = z0 + lz;
  const bool inside = (iy <= n - 1) && (iz <= n - 1);
  const bool own = (iy <= n - 2) && (iz <= n - 2);
  // the out-of-place ops also store the boundary zero at z = n - 1 on padded
  // grids, so their stores cover whole 128-byte lines
  constexpr bool OUT_OF_PLACE = OP != OP_GS;
  const bool zedge = OUT_OF_PLACE && LO > 0 && iy <= n - 2 && iz == n - 1;

  // halo slot (no corners are needed by a 7-point stencil)
  constexpr int NH = 2 * (TY + TZ);
  int hly = 0, hlz = 0;
  if (tid < NH) {
    if (tid < TZ) {
      hly = 0; hlz = tid + 1;
    } else if (tid < 2 * TZ) {
      hly = TY + 1; hlz = tid - TZ + 1;
    } else if (tid < 2 * TZ + TY) {
      hly = tid - 2 * TZ + 1; hlz = 0;
    } else {
      hly = tid - 2 * TZ - TY + 1; hlz = TZ + 1;
    }
  }
  const int hy = y0 - 1 + hly, hz = z0 - 1 + hlz;
  const bool has_halo = (tid < NH) && (hy <= n - 1) && (hz <= n - 1);

  T beta = T(0);
  if (OP == OP_MATVEC) beta = (T)g.scal[prob].beta;
  const bool XD = OP == OP_MATVEC && xdef != nullptr;
  const T alpha_prev = XD ? (T)g.scal[prob].alpha : T(0);
  const T omega1 = (T)g.omega1;

  const int x0 = 1 + xc * g.t.xchunk;
  const int x1 = min(x0 + g.t.xchunk, n - 1);
  using LdT = Ld<T, TI>;
  auto interior = [&](int ix, int jy, int jz) {
    return ix > 0 && ix < n - 1 && jy > 0 && jy < n - 1 && jz > 0 && jz < n - 1;
  };
  auto ldr = [&](int ix, int jy, int jz) -> LdT {
    LdT v{TI(0), T(0)};
    if (x_zero || !interior(ix, jy, jz)) return v;
    const size_t idx = base + ((size_t)ix * n + jy) * LP + jz + LO;
    v.r = in[idx];
    if (OP == OP_MATVEC) v.c = in2[idx];
    if (OP == OP_JAC2Z) v.c = rhs[idx];
    return v;
  };
  auto full = [&](const LdT& v) -> T {
    if (OP == OP_MATVEC) return (T)v.r + beta * v.c;
    if (OP == OP_JACP) return (T)v.r + v.c;
    if (OP == OP_JAC2Z) return (omega1 * v.c) * (T)v.r;
    return (T)v.r;
  };

  // OP_JACP: coarse-plane ring.  Lane l < CSLAB owns slab point
  // (cy0 + l / CZN, cz0 + l % CZN); plane J sits in slot J & 3.  Plane J is
  // stored before the barrier of the first plane whose correction needs it
  // and its global load is issued two planes earlier.
  constexpr int CYN = TY / 2 + 2, CZN = TZ / 2 + 2;
  constexpr int CSLAB = CYN * CZN;
  static_assert(CSLAB <= NT, "coarse slab larger than the workgroup");
  const int nc = (n - 1) / 2 + 1;
  const int cLP = lay_pitch(nc), cLO = lay_off(nc);
  const T* crow = in2 + (size_t)row * (size_t)lay_row(nc);
  const int cy0 = (y0 - 1) >> 1, cz0 = (z0 - 1) >> 1;
  bool cld = false;
  size_t coff = 0;
  if (OP == OP_JACP && tid < CSLAB) {
    const int gy = cy0 + tid / CZN, gz = cz0 + tid % CZN;
    cld = gy <= nc - 1 && gz <= nc - 1;
    coff = (size_t)gy * cLP + gz + cLO;
  }
  auto cload = [&](int J) -> T {
    return (cld && J <= nc - 1) ? crow[(size_t)J * nc * cLP + coff] : T(0);
  };
  auto cstore = [&](int J, T v) {
    if (tid < CSLAB) scs[(J & 3) * CSLAB + tid] = v;
  };
  ProlongLds<T> pco, pch;  // prolongation state of the own and the halo column
  int chi = 0;             // highest coarse plane stored
  T cnext = T(0);          // plane chi + 1, in flight

  auto compS = [&](int jy, int jz, T* S) {
    T cy[KMAX], cz[KMAX];
#pragma unroll
    for (int k = 0; k < KMAX; ++k) {
      cy[k] = (k < K) ? (T)cosT[k * n + jy] : T(0);
      cz[k] = (k < K) ? (T)cosT[k * n + jz] : T(0);
    }
#pragma unroll
    for (int k1 = 0; k1 < KMAX; ++k1) {
      T acc = T(0);
      if (k1 < K) {
#pragma unroll
        for (int k2 = 0; k2 < KMAX; ++k2) {
          if (k2 < K) {
            T t = T(0);
#pragma unroll
            for (int k3 = 0; k3 < KMAX; ++k3)
              if (k3 < K) t += (T)sc[(k1 * K + k2) * K + k3] * cz[k3];
            acc += t * cy[k2];
          }
        }
      }
      S[k1] = acc;
    }
  };
  // reciprocal coefficient 1/a = exp(-log a) at (ix, jy, jz), as stored
  // (bfloat16 bits for the bfloat16 cache, widened by cvt when used)
  using CR = typename std::conditional<CK == 2, uint16_t, T>::type;
  const CR one = CK == 2 ? CR(0x3F80) : CR(1);
  auto coefr = [&](int ix, int jy, int jz, const T* S) -> CR {
    if constexpr (CK == 1) {
      return cache[((size_t)ix * n + jy) * LP + jz + LO];
    } else if constexpr (CK == 2) {
      return cache16[((size_t)ix * n + jy) * LP + jz + LO];
    } else {
      T l = T(0);
#pragma unroll
      for (int k = 0; k < KMAX; ++k)
        if (k < K) l += (T)cosT[k * n + ix] * S[k];
      return dexp(-l);
    }
  };
  auto cvt = [&](CR v) -> T {
    if constexpr (CK == 2)
      return (T)from_bf16(v);
    else
      return v;
  };

  T Sm[KMAX], Sh[KMAX];
#pragma unroll
  for (int k = 0; k < KMAX; ++k) {
    Sm[k] = T(0);
    Sh[k] = T(0);
  }
  if (!CACHED) {
    if (inside) compS(iy, iz, Sm);
    if (has_halo) compS(hy, hz, Sh);
  }

  const T ih2 = (T)g.ih2;

  // Software pipeline: x and 1/a of the own column and of the halo slot are
  // fetched two planes ahead, the right-hand side one plane ahead; loaded
  // values are combined (direction update, prolonged correction, widening)
  // one plane after their loads were issued, so no plane waits on a memory
  // round trip of its own.
  T bm = T(1), bc = T(1);
  LdT xmr{TI(0), T(0)}, xcr{TI(0), T(0)};
  LdT xn{TI(0), T(0)};  // plane x + 1 of the own column, as loaded
  CR bn = one;
  if (inside) {
    xmr = ldr(x0 - 1, iy, iz);
    xcr = ldr(x0, iy, iz);
    xn = ldr(x0 + 1, iy, iz);
    bm = cvt(coefr(x0 - 1, iy, iz, Sm));
    bc = cvt(coefr(x0, iy, iz, Sm));
    bn = coefr(x0 + 1, iy, iz, Sm);
  }
  LdT hcr{TI(0), T(0)}, hn{TI(0), T(0)};
  T hbc = T(1);
  CR hbn = one;
  if (has_halo) {
    hcr = ldr(x0, hy, hz);
    hbc = cvt(coefr(x0, hy, hz, Sh));
    if (x0 + 1 < x1) {
      hn = ldr(x0 + 1, hy, hz);
      hbn = coefr(x0 + 1, hy, hz, Sh);
    }
  }
  // prolonged correction of plane ix of a column (zero where x is)
  auto corr = [&](ProlongLds<T>& pc, int ix, int jy, int jz) -> T {
    const T v = pc.at(scs, CSLAB, ix);
    return (!x_zero && interior(ix, jy, jz)) ? v : T(0);
  };
  if (OP == OP_JACP) {
    const int jlo = (x0 - 1) >> 1;
    chi = (x0 + 3) >> 1;
    for (int J = jlo; J <= chi; ++J) cstore(J, cload(J));
    cnext = cload(chi + 1);
    __syncthreads();
    if (inside) {
      pco.init(scs, CSLAB, CZN, cy0, cz0, iy, iz, x0 - 1);
      xmr.c = corr(pco, x0 - 1, iy, iz);
      xcr.c = corr(pco, x0, iy, iz);
      xn.c = corr(pco, x0 + 1, iy, iz);
    }
    if (has_halo) {
      pch.init(scs, CSLAB, CZN, cy0, cz0, hy, hz, x0);
      hcr.c = corr(pch, x0, hy, hz);
      if (x0 + 1 < x1) hn.c = corr(pch, x0 + 1, hy, hz);
    }
  }
  T xm = full(xmr), xcur = full(xcr), hcur = full(hcr);
  T fxm = face(bm, bc);
  constexpr bool USES_B =
      (OP == OP_RESID || OP == OP_GS || OP == OP_JAC || OP == OP_JACP || OP == OP_JAC2Z);
  T bv = T(0);
  if (USES_B && own) bv = rhs[base + ((size_t)x0 * n + iy) * LP + iz + LO];
  // deferred step: the iterate one plane ahead, the old direction as loaded
  T xv = T(0), pold = T(0);
  if (OP == OP_MATVEC) {
    pold = xcr.c;
    if (XD && own) xv = xdef[base + ((size_t)x0 * n + iy) * LP + iz + LO];
  }
  double dot = 0.0;
  const int cidx = (ly + 1) * PZ + (lz + 1);
  const int hidx = hly * PZ + hlz;

  for (int ix = x0; ix < x1; ++ix) {
    const int buf = ix & 1;
    // prefetch: plane ix+2 of the columns, plane ix+1 of the right-hand side
    const bool own_next = inside && ix + 2 <= n - 1;
    const bool halo_next = has_halo && ix + 2 < x1;
    LdT xnn{TI(0), T(0)}, hnn{TI(0), T(0)};
    CR bnn = one, hbnn = one;
    T bvn = T(0);
    if (own_next) {
      xnn = ldr(ix + 2, iy, iz);
      bnn = coefr(ix + 2, iy, iz, Sm);
    }
    if (halo_next) {
      hnn = ldr(ix + 2, hy, hz);
      hbnn = coefr(ix + 2, hy, hz, Sh);
    }
    if (USES_B && own && ix + 1 < x1) bvn = __builtin_nontemporal_load(&rhs[base + ((size_t)(ix + 1) * n + iy) * LP + iz + LO]);
    T xvn = T(0);
    if (XD && own && ix + 1 < x1) xvn = xdef[base + ((size_t)(ix + 1) * n + iy) * LP + iz + LO];
    if (OP == OP_JACP && ((ix + 3) >> 1) > chi) {
      ++chi;
      cstore(chi, cnext);
      cnext = cload(chi + 1);
    }
    sx[buf][cidx] = inside ? xcur : T(0);
    sb[buf][cidx] = inside ? bc : T(1);
    if (tid < NH) {
      sx[buf][hidx] = has_halo ? hcur : T(0);
      sb[buf][hidx] = has_halo ? hbc : T(1);
    }
    __syncthreads();
    if (OP == OP_JACP) {
      if (own_next) xnn.c = corr(pco, ix + 2, iy, iz);
      if (halo_next) hnn.c = corr(pch, ix + 2, hy, hz);
    }
    const T xp = full(xn);
    const T bp = cvt(bn);
    const T fxp = face(bc, bp);
    if (own || zedge) {
      const T xym = sx[buf][cidx - PZ], xyp = sx[buf][cidx + PZ];
      const T xzm = sx[buf][cidx - 1], xzp = sx[buf][cidx + 1];
      const T fym = face(bc, sb[buf][cidx - PZ]), fyp = face(bc, sb[buf][cidx + PZ]);
      const T fzm = face(bc, sb[buf][cidx - 1]), fzp = face(bc, sb[buf][cidx + 1]);
      const T diag = ((fxm + fxp) + (fym + fyp)) + (fzm + fzp);
      const T off = ((fxm * xm + fxp * xp) + (fym * xym + fyp * xyp)) + (fzm * xzm + fzp * xzp);
      const size_t idx = base + ((size_t)ix * n + iy) * LP + iz + LO;
      // the z = n - 1 lane computes from in-bounds (zero-start) values and
      // stores a zero in the same vector store as its line's vertices
      if (OP == OP_RESID) {
        const T r = bv - ih2 * (diag * xcur - off);
        if (out) __builtin_nontemporal_store(own ? r : T(0), &out[idx]);
        if (partial && own) dot += (double)r * (double)r;
      } else if (OP == OP_MATVEC) {
        const T q = own ? ih2 * (diag * xcur - off) : T(0);
        __builtin_nontemporal_store(q, &out[idx]);
        __builtin_nontemporal_store(xcur, &out2[idx]);
        if (XD) __builtin_nontemporal_store(own ? xv + alpha_prev * pold : T(0), &xdef[idx]);
        dot += (double)xcur * (double)q;
      } else if (OP == OP_JAC || OP == OP_JACP || OP == OP_JAC2Z) {
        const T v = xcur + omega * (bv - ih2 * (diag * xcur - off)) * drcp(ih2 * diag);
        const T val = own ? v : T(0);
        __builtin_nontemporal_store(val, &out[idx]);
        if (partial) dot += (double)bv * (double)val;
      } else {  // OP_GS
        T val = xcur;
        const bool upd = ((ix + iy + iz) & 1) == color;
        if (upd) {
          const T gs = (bv + ih2 * off) * drcp(ih2 * diag);
          val = xcur + omega * (gs - xcur);
          out[idx] = val;
        } else if (x_zero) {
          val = T(0);
          out[idx] = val;
        }
        if (partial) {
          const T bb = upd ? bv : rhs[idx];
          dot += (double)bb * (double)val;
        }
      }
    }
    xm = xcur;
    xcur = xp;
    if (OP == OP_MATVEC) {
      pold = xn.c;
      xv = xvn;
    }
    xn = xnn;
    bm = bc;
    bc = bp;
    bn = bnn;
    fxm = fxp;
    hcur = full(hn);
    hbc = cvt(hbn);
    hn = hnn;
    hbn = hbnn;
    bv = bvn;
  }
  const bool want = (OP == OP_MATVEC) || (OP == OP_RESID && partial != nullptr) ||
                    ((OP == OP_GS || OP == OP_JAC || OP == OP_JACP) && partial != nullptr &&
                     prob >= top_begin);
  if (want) {
    const double s = block_sum<NT>(dot, lds.sred, tid);
    if (tid == 0) partial[poff[prob] + tile] = s;
  }
}

template <typename T, typename TI, int TY, int TZ, int OP, int CK>
__global__ void __launch_bounds__(TY* TZ)
    k_march(GridArgs g, const TI* in, const T* in2, const T* rhs, T* out, T* out2,
            const int* __restrict__ poff, double* __restrict__ partial, int color,
            int x_zero, int top_begin, T omega, T* __restrict__ xdef) {
  __shared__ MarchLds<T, TY, TZ, OP, CK> lds;
  march_tile<T, TI, TY, TZ, OP, CK>(lds, g, xcd_swizzle(blockIdx.x, gridDim.x), threadIdx.x, in,
                                    in2, rhs, out, out2, poff, partial, color, x_zero, top_begin,
                                    omega, xdef);
}

// One FP64 op over the rows of several groups (grids of different size, cached
// coefficient) in one launch: a small group's launch takes the latency of one
// march on a nearly idle chip, and these run side by side.  Workgroups have the
// 512 threads of the largest tile and take several smaller tiles at once.  A
// tile is whole waves with LDS of its own, and only its own waves read what they
// write; waves of a tile that ends early (an inactive problem, a shorter last
// chunk) leave, and tiles may stand at different barriers of the code.  That rests
// on the machine's barrier, not on the language's: s_barrier counts the waves of a
// workgroup that arrive, at whichever s_barrier, and those that ended, so the waves
// of one tile pass each of theirs together.  A group's workgroups start at a
// multiple of 8, which keeps its tiles in XCD order.
// With the residual update likewise (k_groups): a 17^3..65^3 law estimate 4.92 ->
// 4.52 ms, graph replay of a 64/16/4 estimate 2.32 -> 1.96, an objective up to
// 65^3 3.23 -> 2.89, an adaptive step up to 257^3 26.4 -> 24.9; full batches gain
// the tails of the smaller groups (9^3..129^3 FP64 57.7 -> 56.6 ms).
constexpr int GM_THREADS = 512;

template <typename TI, int OP, int TY, int TZ>
__device__ __forceinline__ void march_group(char* smem, const MarchGroup& m, int wg,
                                            const int* poff, double* partial) {
  constexpr int NT = TY * TZ, PACK = GM_THREADS / NT;
  using Lds = MarchLds<double, TY, TZ, OP, 1>;
  const int tiles = m.g.rows * m.g.t.tiles_per_row, wgs = (tiles + PACK - 1) / PACK;
  if (wg >= wgs) return;
  const int sub = __builtin_amdgcn_readfirstlane(threadIdx.x / NT);
  const int bid = xcd_swizzle(wg, wgs) * PACK + sub;
  if (bid >= tiles) return;
  march_tile<double, TI, TY, TZ, OP, 1>(reinterpret_cast<Lds*>(smem)[sub], m.g, bid,
                                        threadIdx.x - sub * NT, (const TI*)m.in, m.in2, m.rhs,
                                        m.out, m.out2, poff, partial, 0, 0, 0, 1.0, m.xdef);
}

template <typename TI, int OP>
__global__ void __launch_bounds__(GM_THREADS)
    k_march_groups(MarchTable t, const int* __restrict__ poff, double* __restrict__ partial) {
  constexpr size_t L64 = sizeof(MarchLds<double, 8, 64, OP, 1>);
  constexpr size_t L32 = 2 * sizeof(MarchLds<double, 8, 32, OP, 1>);
  constexpr size_t L16 = 2 * sizeof(MarchLds<double, 16, 16, OP, 1>);
  constexpr size_t L8 = 8 * sizeof(MarchLds<double, 8, 8, OP, 1>);
  constexpr size_t LA = L64 > L32 ? L64 : L32, LB = L16 > L8 ? L16 : L8;
  __shared__ __align__(16) char smem[LA > LB ? LA : LB];
  int i = 0;
  while (i + 1 < t.count && (int)blockIdx.x >= t.gr[i + 1].begin) ++i;
  const MarchGroup& m = t.gr[i];
  const int wg = (int)blockIdx.x - m.begin;
  if (m.g.t.TZ == 64)
    march_group<TI, OP, 8, 64>(smem, m, wg, poff, partial);
  else if (m.g.t.TZ == 32)
    march_group<TI, OP, 8, 32>(smem, m, wg, poff, partial);
  else if (m.g.t.TZ == 16)
    march_group<TI, OP, 16, 16>(smem, m, wg, poff, partial);
  else
    march_group<TI, OP, 8, 8>(smem, m, wg, poff, partial);
}

template <typename TI, int OP>
static void launch_march_groups(MarchTable& t, const int* poff, double* partial, hipStream_t s) {
  int wg = 0;
  for (int i = 0; i < t.count; ++i) {
    MarchGroup& m = t.gr[i];
    m.begin = wg;
    const int pack = GM_THREADS / (m.g.t.TY * m.g.t.TZ);
    wg += (cdiv((long long)m.g.rows * m.g.t.tiles_per_row, pack) + 7) & ~7;
  }
  if (wg > 0)
    hipLaunchKernelGGL((k_march_groups<TI, OP>), dim3(wg), dim3(GM_THREADS), 0, s, t, poff, partial);
}
void matvec_groups(MarchTable& t, bool z32, const int* poff, double* partial, hipStream_t s) {
  if (z32)
    launch_march_groups<float, OP_MATVEC>(t, poff, partial, s);
  else
    launch_march_groups<double, OP_MATVEC>(t, poff, partial, s);
}
void resid_groups(MarchTable& t, const int* poff, double* partial, hipStream_t s) {
  launch_march_groups<double, OP_RESID>(t, poff, partial, s);
}


template <typename T, typename TI, int OP, int CK>
static void launch_march2(const GridArgs& g, const TI* in, const T* in2, const T* rhs, T* out,
                          T* out2, const int* poff, double* partial, int color, int x_zero,
                          int top_begin, T omega, hipStream_t s, T* xdef) {
  const int nblk = g.rows * g.t.tiles_per_row;
#define MLSGD_LAUNCH(TY_, TZ_)                                                              \
  hipLaunchKernelGGL((k_march<T, TI, TY_, TZ_, OP, CK>), dim3(nblk), dim3(TY_ * TZ_), 0, s, \
                     g, in, in2, rhs, out, out2, poff, partial, color, x_zero, top_begin, omega, \
                     xdef)
  if (g.t.TZ == 8) {
    MLSGD_LAUNCH(8, 8);
  } else if (g.t.TZ == 16) {
    MLSGD_LAUNCH(16, 16);
  } else if (g.t.TZ == 32) {
    MLSGD_LAUNCH(8, 32);
  } else if (g.t.TY == 8) {
    MLSGD_LAUNCH(8, 64);
  } else if (g.t.TY == 16) {
    MLSGD_LAUNCH(16, 64);
  } else {
    MLSGD_LAUNCH(4, 64);
  }
#undef MLSGD_LAUNCH
}

template <typename T, typename TI, int OP>
static void launch_march(const GridArgs& g, const TI* in, const T* in2, const T* rhs, T* out,
                         T* out2, const int* poff, double* partial, int color, int x_zero,
                         int top_begin, T omega, hipStream_t s, T* xdef = nullptr) {
  if (g.rows <= 0) return;
  if (!g.cache)
    launch_march2<T, TI, OP, 0>(g, in, in2, rhs, out, out2, poff, partial, color, x_zero,
                                top_begin, omega, s, xdef);
  else if (sizeof(T) == 4 && g.cache_bf16)
    launch_march2<T, TI, OP, 2>(g, in, in2, rhs, out, out2, poff, partial, color, x_zero,
                                top_begin, omega, s, xdef);
  else
    launch_march2<T, TI, OP, 1>(g, in, in2, rhs, out, out2, poff, partial, color, x_zero,
                                top_begin, omega, s, xdef);
}

template <typename T>
void march_resid(const GridArgs& g, const T* x, const T* b, T* r, hipStream_t s) {
  launch_march<T, T, OP_RESID>(g, x, nullptr, b, r, nullptr, nullptr, nullptr, 0, 0, 0, T(1), s);
}
void march_resid_norm(const GridArgs& g, const double* x, const double* b, const int* poff,
                      double* partial, hipStream_t s) {
  launch_march<double, double, OP_RESID>(g, x, nullptr, b, nullptr, nullptr, poff, partial, 0, 0,
                                         0, 1.0, s);
}
template <typename T, typename TZ>
void march_matvec(const GridArgs& g, const TZ* z, const T* p_old, T* p_new, T* q,
                  const int* poff, double* partial, hipStream_t s, T* x) {
  launch_march<T, TZ, OP_MATVEC>(g, z, p_old, nullptr, q, p_new, poff, partial, 0, 0, 0, T(1), s,
                                 x);
}
template <typename T>
void march_gs(const GridArgs& g, T* x, const T* b, int color, int x_zero, const int* poff,
              double* partial, int top_begin, double omega, hipStream_t s) {
  launch_march<T, T, OP_GS>(g, x, nullptr, b, x, nullptr, poff, partial, color, x_zero, top_begin,
                            (T)omega, s);
}
template void march_resid<double>(const GridArgs&, const double*, const double*, double*,
                                  hipStream_t);
template void march_resid<float>(const GridArgs&, const float*, const float*, float*,
                                 hipStream_t);
template void march_matvec<double, double>(const GridArgs&, const double*, const double*,
                                           double*, double*, const int*, double*, hipStream_t,
                                           double*);
template void march_matvec<double, float>(const GridArgs&, const float*, const double*, double*,
                                          double*, const int*, double*, hipStream_t, double*);
template void march_gs<double>(const GridArgs&, double*, const double*, int, int, const int*,
                               double*, int, double, hipStream_t);
template void march_gs<float>(const GridArgs&, float*, const float*, int, int, const int*,
                              double*, int, double, hipStream_t);
template <typename T>
void march_jac(const GridArgs& g, const T* xin, const T* xc, const T* b, T* xout, int x_zero,
               double omega, const int* poff, double* partial, int top_begin, hipStream_t s) {
  if (xc && !x_zero)
    launch_march<T, T, OP_JACP>(g, xin, xc, b, xout, nullptr, poff, partial, 0, 0, top_begin,
                                (T)omega, s);
  else
    launch_march<T, T, OP_JAC>(g, xin, nullptr, b, xout, nullptr, poff, partial, 0, x_zero,
                               top_begin, (T)omega, s);
}
template void march_jac<double>(const GridArgs&, const double*, const double*, const double*,
                                double*, int, double, const int*, double*, int, hipStream_t);
template void march_jac<float>(const GridArgs&, const float*, const float*, const float*, float*,
                               int, double, const int*, double*, int, hipStream_t);

static int grid_for(long long total, int bs);

template <typename T>
void march_jac2z(const GridArgs& g, const T* dinv, const T* b, T* xout, double omega1,
                 double omega2, hipStream_t s) {
  GridArgs g2 = g;
  g2.omega1 = omega1;
  launch_march<T, T, OP_JAC2Z>(g2, dinv, nullptr, b, xout, nullptr, nullptr, nullptr, 0, 0, 0,
                               (T)omega2, s);
}
template void march_jac2z<double>(const GridArgs&, const double*, const double*, double*, double,
                                  double, hipStream_t);
template void march_jac2z<float>(const GridArgs&, const float*, const float*, float*, double,
                                 double, hipStream_t);

// ---------------------------------------------------------------------------
// Fused pre-smoothing and residual.  From x = 0, the first two Chebyshev
// steps and the residual of their result in one pass:
//   x1 = omega1 b / D                   (pointwise, from b and the stored 1/D)
//   x2 = x1 + omega2 D^-1 (b - A x1)
//   r  = b - A x2
// x2 and r are written; b, 1/D and 1/a are read once: 40 B per point instead
// of 32 + 32 for the two-step pass and a residual pass.  Neighbours and
// summation order are those two passes'; faces and 1/D of the steps come
// from the one-step reciprocal srcp (within a few ulp of theirs in FP64).
//
// The march lags the residual one plane behind the second step.  At plane q
// the workgroup puts x1 and 1/a of its patch and a two-point ring in LDS,
// forms x2 on the patch and its one-point ring (LDS, double-buffered), and
// then r on plane q - 1.  Besides its patch column, thread t owns one ring
// slot: t < NR a column of the one-point ring (x2 is formed there, so it
// keeps x1 and 1/a of three planes like the patch columns), NR <= t < 2 NR a
// slot of the two-point ring, and the next four threads the corners of the
// one-point ring (NR = 2 (TY + TZ); the corners of the two-point ring are not
// needed).  1/a sits in a ring of three LDS planes, as plane q - 1 is still
// read after the next plane is stored.  Each patch column keeps the faces it
// formed for x2 on plane q and reuses them for r on that plane one step
// later.  The loads of plane q + 2 are issued at the start of step q and
// combined at its end.
//
// RH: instead of r, the x part of the full-weighting restriction of r,
//   h(I) = r(2I-1) / 4 + r(2I) / 2 + r(2I+1) / 4   (per interior column)
// goes into plane I of rout, for the coarse planes I with x0 < 2I < x1 of
// the workgroup's x chunk (x0 odd: one chunk, or chunks of even length), so
// every coarse plane is written by one chunk; the march forms r on one more
// plane (x1) for the last of them.  k_restrict_yz_rows finishes the
// restriction from h: 28 instead of 32 B per fine point for the pass and
// the restriction's read.
// ---------------------------------------------------------------------------
template <typename T, int TY, int TZ, int CK, bool RH>
__global__ void __launch_bounds__(TY* TZ)
    k_pre2r(GridArgs g, const T* __restrict__ dinv, const T* __restrict__ rhs,
            T* __restrict__ xout, T* __restrict__ rout, T omega1, T omega2) {
  constexpr int NT = TY * TZ;
  constexpr int PZ = TZ + 4;
  constexpr int PLANE = (TY + 4) * PZ;
  constexpr int NR = 2 * (TY + TZ);
  static_assert(2 * NR + 4 <= NT, "tile too small for its rings");
  using CR = typename std::conditional<CK == 2, uint16_t, T>::type;
  __shared__ T s1[PLANE];      // x1, plane q
  __shared__ T sb[3][PLANE];   // 1/a, plane q in slot q % 3
  __shared__ T s2[2][PLANE];   // x2, plane q in slot q & 1

  const int n = g.n;
  const int LP = lay_pitch(n), LO = lay_off(n);
  const int bid = xcd_swizzle(blockIdx.x, gridDim.x);
  const int tpr = g.t.tiles_per_row;
  const int row = bid / tpr;
  const int tile = bid - row * tpr;
  int tt = tile;
  const int ty = tt % g.t.nty;
  tt /= g.t.nty;
  const int tz = tt % g.t.ntz;
  const int xc = tt / g.t.ntz;
  const int prob = g.row0 + row;
  if (g.scal && !g.scal[prob].active) return;  // uniform per workgroup

  const size_t base = (size_t)row * (size_t)g.stride;
  const CR* __restrict__ cache = (const CR*)g.cache + (size_t)prob * (size_t)g.stride;
  const int tid = threadIdx.x;
  const int y0 = 1 + ty * TY, z0 = 1 + tz * TZ;
  const T ih2 = (T)g.ih2;

  // LDS coordinates: the patch is [2, TY+2) x [2, TZ+2); grid vertex (jy, jz)
  // sits at (jy - y0 + 2, jz - z0 + 2)
  auto ring_slot = [&](int t, int d) {  // slot t < NR of the d-point ring
    int a, b;
    if (t < TZ) {
      a = 2 - d; b = 2 + t;
    } else if (t < 2 * TZ) {
      a = TY + 1 + d; b = 2 + t - TZ;
    } else if (t < 2 * TZ + TY) {
      a = 2 + t - 2 * TZ; b = 2 - d;
    } else {
      a = 2 + t - 2 * TZ - TY; b = TZ + 1 + d;
    }
    return a * PZ + b;
  };
  const int ly = tid / TZ, lz = tid - (tid / TZ) * TZ;
  const int oidx = (ly + 2) * PZ + (lz + 2);
  int sidx = 0;
  const bool ring1 = tid < NR;                       // x2 is formed at this slot
  const bool s_on = tid < 2 * NR + 4;
  if (tid < NR) {
    sidx = ring_slot(tid, 1);
  } else if (tid < 2 * NR) {
    sidx = ring_slot(tid - NR, 2);
  } else if (s_on) {
    const int k = tid - 2 * NR;
    sidx = ((k >> 1) ? TY + 2 : 1) * PZ + ((k & 1) ? TZ + 2 : 1);
  }
  const int oy = y0 - 2 + oidx / PZ, oz = z0 - 2 + oidx % PZ;
  const int sy = y0 - 2 + sidx / PZ, sz = z0 - 2 + sidx % PZ;
  auto in_int = [&](int jy, int jz) { return jy >= 1 && jz >= 1 && jy <= n - 2 && jz <= n - 2; };
  const bool o_int = in_int(oy, oz);
  const bool s_int = s_on && in_int(sy, sz);

  // one plane of one column as loaded: b, 1/D (interior only) and 1/a
  struct Raw {
    T b, d;
    CR a;
  };
  const CR one = CK == 2 ? CR(0x3F80) : CR(1);
  // Columns are addressed as in k_post2: a 32-bit element offset in plane 0
  // and the plane stride, every in-grid vertex loaded without a mask (b and
  // 1/D are zero off the interior, so x1 is too), ring slots outside the
  // grid reading the nearest in-grid column (their values only reach
  // discarded non-interior results).
  const T* __restrict__ brow = rhs + base;
  const T* __restrict__ drow = dinv + base;
  const uint32_t pstr = (uint32_t)n * (uint32_t)LP;
  auto col_off = [&](int jy, int jz) -> uint32_t {
    jy = min(max(jy, 0), n - 1);
    jz = min(max(jz, 0), n - 1);
    return (uint32_t)(jy * LP + jz + LO);
  };
  const uint32_t ooff = col_off(oy, oz);
  const uint32_t soff = col_off(sy, sz);
  auto load = [&](int ix, uint32_t off) -> Raw {
    Raw v{T(0), T(0), one};
    if (ix < 0 || ix > n - 1) return v;   // uniform
    const size_t e = (size_t)off + (size_t)ix * pstr;
    v.a = cache[e];
    v.b = brow[e];
    v.d = drow[e];
    return v;
  };
  auto cvt = [&](CR v) -> T {
    if constexpr (CK == 2)
      return (T)from_bf16(v);
    else
      return v;
  };
  auto x1of = [&](const Raw& v) -> T { return (omega1 * v.b) * v.d; };

  const int x0 = 1 + xc * g.t.xchunk;
  const int x1 = min(x0 + g.t.xchunk, n - 1);
  // last step: r on plane x1 as well when the restriction reads it
  const int qend = RH ? min(x1 + 1, n - 1) : x1;

  // On entry to step q: x1 and 1/a at q-1, q, q+1 and b at q, q+1 for the
  // patch column (o*) and the slot (s*; two-point ring slots and corners use
  // plane q only)
  T oxm, oxc, oxp, obm, obc, obp, orc, orp;
  T sxm = T(0), sxc = T(0), sxp = T(0), sbm = T(1), sbc = T(1), sbp = T(1), src = T(0), srp = T(0);
  {
    const int q = x0 - 1;
    const Raw m = load(q - 1, ooff), c = load(q, ooff),
              p = load(q + 1, ooff);
    oxm = x1of(m); oxc = x1of(c); oxp = x1of(p);
    obm = cvt(m.a); obc = cvt(c.a); obp = cvt(p.a);
    orc = c.b; orp = p.b;
    if (s_on) {
      const Raw sm = load(q - 1, soff), sc = load(q, soff),
                sp = load(q + 1, soff);
      sxm = x1of(sm); sxc = x1of(sc); sxp = x1of(sp);
      sbm = cvt(sm.a); sbc = cvt(sc.a); sbp = cvt(sp.a);
      src = sc.b; srp = sp.b;
    }
  }

  // patch column: x2 at q-2, q-1, the faces of plane q-1 and b at q-1; with
  // RH the partial h of the coarse plane being summed
  T x2a = T(0), x2b = T(0), rm_ = T(0), hacc = T(0);
  T gfxm = T(0), gfxp = T(0), gfym = T(0), gfyp = T(0), gfzm = T(0), gfzp = T(0), gdiag = T(1);

  for (int q = x0 - 1; q <= qend; ++q) {
    const Raw on = load(q + 2, ooff);
    Raw sn{T(0), T(0), one};
    if (s_on) sn = load(q + 2, soff);

    T* __restrict__ b3 = sb[q % 3];
    s1[oidx] = oxc;
    b3[oidx] = obc;
    if (s_on) {
      s1[sidx] = sxc;
      b3[sidx] = sbc;
    }
    __syncthreads();

    // x2 on plane q: patch and one-point ring
    const bool qin = q >= 1 && q <= n - 2;
    T x2c = T(0);
    T fxm = T(0), fxp = T(0), fym = T(0), fyp = T(0), fzm = T(0), fzp = T(0), diag = T(1);
    if (qin && o_int) {
      fxm = sface(obc, obm);
      fxp = sface(obc, obp);
      fym = sface(obc, b3[oidx - PZ]);
      fyp = sface(obc, b3[oidx + PZ]);
      fzm = sface(obc, b3[oidx - 1]);
      fzp = sface(obc, b3[oidx + 1]);
      diag = ((fxm + fxp) + (fym + fyp)) + (fzm + fzp);
      const T off = ((fxm * oxm + fxp * oxp) + (fym * s1[oidx - PZ] + fyp * s1[oidx + PZ])) +
                    (fzm * s1[oidx - 1] + fzp * s1[oidx + 1]);
      x2c = oxc + omega2 * (orc - ih2 * (diag * oxc - off)) * srcp(ih2 * diag);
    }
    T* __restrict__ x2s = s2[q & 1];
    x2s[oidx] = x2c;
    if (ring1) {
      T v = T(0);
      if (qin && s_int) {
        const T hxm = sface(sbc, sbm), hxp = sface(sbc, sbp);
        const T hym = sface(sbc, b3[sidx - PZ]), hyp = sface(sbc, b3[sidx + PZ]);
        const T hzm = sface(sbc, b3[sidx - 1]), hzp = sface(sbc, b3[sidx + 1]);
        const T hd = ((hxm + hxp) + (hym + hyp)) + (hzm + hzp);
        const T hoff = ((hxm * sxm + hxp * sxp) + (hym * s1[sidx - PZ] + hyp * s1[sidx + PZ])) +
                       (hzm * s1[sidx - 1] + hzp * s1[sidx + 1]);
        v = sxc + omega2 * (src - ih2 * (hd * sxc - hoff)) * srcp(ih2 * hd);
      }
      x2s[sidx] = v;
    }
    __syncthreads();

    // r on plane q-1 from x2 of planes q-2, q-1 (LDS with ring), q
    const int qr = q - 1;
    if (qr >= x0 && o_int) {
      const T* __restrict__ x2p = s2[qr & 1];
      const T off = ((gfxm * x2a + gfxp * x2c) + (gfym * x2p[oidx - PZ] + gfyp * x2p[oidx + PZ])) +
                    (gfzm * x2p[oidx - 1] + gfzp * x2p[oidx + 1]);
      const T r = rm_ - ih2 * (gdiag * x2b - off);
      const size_t e = base + ((size_t)qr * n + oy) * LP + oz + LO;
      if constexpr (RH) {
        if (qr < x1) __builtin_nontemporal_store(x2b, &xout[e]);
        if (qr & 1) {
          // r(qr) closes coarse plane (qr - 1) / 2 and opens (qr + 1) / 2
          if (qr >= x0 + 2) {
            const size_t eh = base + ((size_t)((qr - 1) >> 1) * n + oy) * LP + oz + LO;
            __builtin_nontemporal_store(hacc + T(0.25) * r, &rout[eh]);
          }
          hacc = T(0.25) * r;
        } else {
          hacc = hacc + T(0.5) * r;
        }
      } else {
        __builtin_nontemporal_store(x2b, &xout[e]);
        __builtin_nontemporal_store(r, &rout[e]);
      }
    }

    // advance one plane
    x2a = x2b;
    x2b = x2c;
    rm_ = orc;
    gfxm = fxm; gfxp = fxp; gfym = fym; gfyp = fyp; gfzm = fzm; gfzp = fzp; gdiag = diag;
    oxm = oxc; oxc = oxp; oxp = x1of(on);
    obm = obc; obc = obp; obp = cvt(on.a);
    orc = orp; orp = on.b;
    if (s_on) {
      sxm = sxc; sxc = sxp; sxp = x1of(sn);
      sbm = sbc; sbc = sbp; sbp = cvt(sn.a);
      src = srp; srp = sn.b;
    }
  }
}

// ---------------------------------------------------------------------------
// Fused post-smoothing: two Chebyshev steps after the coarse-grid correction
// in one pass,
//   y  = x + P e                        (trilinear prolongation of the coarse e)
//   x3 = y  + omega_a D^-1 (b - A y)
//   x4 = x3 + omega_b D^-1 (b - A x3)
// with the partial sums of <b, x4> for the problems whose top grid this is.
// x, e / 8, b and 1/a are read and x4 written once: 33 B per point instead of
// 33 + 32 for the step with the folded correction and a plain step.  Both
// steps use k_march's neighbours and summation order, with faces and 1/D from
// srcp as in k_pre2r.
//
// The plane pipeline is that of k_pre2r (y in place of x1): y and 1/a of the
// patch and a two-point ring on plane q in LDS, x3 on the patch and its
// one-point ring, x4 on plane q - 1.  The coarse planes covering the
// two-point ring's footprint sit in a four-plane LDS ring (TY/2 + 3 by
// TZ/2 + 3 coarse points); every column forms its prolonged correction with
// ProlongLds, two planes ahead of its use.  Every stencil column forms its
// face to +x once and keeps the one to -x from the plane before.  In FP64
// the faces to +y and +z are also formed once per position and plane, into
// LDS (three plane slots, from 1/a stored one plane ahead), so both stencils
// read their y and z faces instead of forming them; in FP32, whose
// reciprocal is one instruction, they are formed from 1/a where used (a
// three-plane 1/a ring), which measured faster.
//
// XZ: x is zero and not read (y = P e, 25 B per point), for the
// pre-smoothing of a full-multigrid cycle from the prolonged solution of the
// grid below.
// ---------------------------------------------------------------------------
template <typename T, int TY, int TZ, int CK, bool XZ>
__global__ void __launch_bounds__(TY* TZ)
    k_post2(GridArgs g, const T* __restrict__ xin, const T* __restrict__ xc,
            const T* __restrict__ rhs, T* __restrict__ xout, const int* __restrict__ poff,
            double* __restrict__ partial, int top_begin, T omega_a, T omega_b) {
  constexpr int NT = TY * TZ;
  constexpr int PZ = TZ + 4;
  constexpr int PLANE = (TY + 4) * PZ;
  constexpr int NR = 2 * (TY + TZ);
  static_assert(2 * NR + 4 <= NT, "tile too small for its rings");
  constexpr int CYN = TY / 2 + 3, CZN = TZ / 2 + 3;
  constexpr int CSLAB = CYN * CZN;
  static_assert(CSLAB <= NT, "coarse slab larger than the workgroup");
  using CR = typename std::conditional<CK == 2, uint16_t, T>::type;
  // FP64 shares faces through LDS (its reciprocal costs three operations);
  // FP32 forms every face from 1/a (one reciprocal instruction)
  constexpr bool SHARE = sizeof(T) == 8;
  constexpr int NF = SHARE ? 3 : 1, NB = SHARE ? 1 : 3;
  __shared__ T s1[PLANE];      // y, plane q
  __shared__ T sb[NB][PLANE];  // 1/a: plane q + 1 (SHARE) or plane q in slot q % 3
  __shared__ T fy[NF][SHARE ? PLANE : 1];  // face to +y, plane p in slot p % 3
  __shared__ T fz[NF][SHARE ? PLANE : 1];  // face to +z, plane p in slot p % 3
  __shared__ T s3[2][PLANE];   // x3, plane q in slot q & 1
  __shared__ T scs[4 * CSLAB]; // coarse plane J in slot J & 3
  __shared__ double sred[NT / 64];

  const int n = g.n;
  const int LP = lay_pitch(n), LO = lay_off(n);
  const int bid = xcd_swizzle(blockIdx.x, gridDim.x);
  const int tpr = g.t.tiles_per_row;
  const int row = bid / tpr;
  const int tile = bid - row * tpr;
  int tt = tile;
  const int ty = tt % g.t.nty;
  tt /= g.t.nty;
  const int tz = tt % g.t.ntz;
  const int xcix = tt / g.t.ntz;
  const int prob = g.row0 + row;
  if (g.scal && !g.scal[prob].active) return;  // uniform per workgroup

  const size_t base = (size_t)row * (size_t)g.stride;
  const CR* __restrict__ cache = (const CR*)g.cache + (size_t)prob * (size_t)g.stride;
  const int tid = threadIdx.x;
  const int y0 = 1 + ty * TY, z0 = 1 + tz * TZ;
  const T ih2 = (T)g.ih2;

  auto ring_slot = [&](int t, int d) {  // slot t < NR of the d-point ring
    int a, b;
    if (t < TZ) {
      a = 2 - d; b = 2 + t;
    } else if (t < 2 * TZ) {
      a = TY + 1 + d; b = 2 + t - TZ;
    } else if (t < 2 * TZ + TY) {
      a = 2 + t - 2 * TZ; b = 2 - d;
    } else {
      a = 2 + t - 2 * TZ - TY; b = TZ + 1 + d;
    }
    return a * PZ + b;
  };
  const int ly = tid / TZ, lz = tid - (tid / TZ) * TZ;
  const int oidx = (ly + 2) * PZ + (lz + 2);
  int sidx = 0;
  const bool ring1 = tid < NR;
  const bool s_on = tid < 2 * NR + 4;
  if (tid < NR) {
    sidx = ring_slot(tid, 1);
  } else if (tid < 2 * NR) {
    sidx = ring_slot(tid - NR, 2);
  } else if (s_on) {
    const int k = tid - 2 * NR;
    sidx = ((k >> 1) ? TY + 2 : 1) * PZ + ((k & 1) ? TZ + 2 : 1);
  }
  const int oy = y0 - 2 + oidx / PZ, oz = z0 - 2 + oidx % PZ;
  const int sy = y0 - 2 + sidx / PZ, sz = z0 - 2 + sidx % PZ;
  auto in_int = [&](int jy, int jz) { return jy >= 1 && jz >= 1 && jy <= n - 2 && jz <= n - 2; };
  const bool o_int = in_int(oy, oz);
  const bool s_int = s_on && in_int(sy, sz);

  struct Raw {  // one plane of one column as loaded: x, b (interior only), 1/a
    T x, b;
    CR a;
  };
  const CR one = CK == 2 ? CR(0x3F80) : CR(1);
  // A column is addressed by its 32-bit element offset in plane 0 and the
  // plane stride.  Every in-grid vertex is loaded without a mask: boundary
  // vertices and padding hold zeros in x and b, and the prolonged coarse
  // correction vanishes on the boundary.  Ring slots outside the grid read
  // the nearest in-grid column; their values feed only results at
  // non-interior positions, which are set to zero or discarded.
  const T* __restrict__ xrow = XZ ? nullptr : xin + base;
  const T* __restrict__ brow = rhs + base;
  const uint32_t pstr = (uint32_t)n * (uint32_t)LP;
  auto col_off = [&](int jy, int jz) -> uint32_t {
    jy = min(max(jy, 0), n - 1);
    jz = min(max(jz, 0), n - 1);
    return (uint32_t)(jy * LP + jz + LO);
  };
  const uint32_t ooff = col_off(oy, oz);
  const uint32_t soff = col_off(sy, sz);
  auto load = [&](int ix, uint32_t off) -> Raw {
    Raw v{T(0), T(0), one};
    if (ix < 0 || ix > n - 1) return v;   // uniform
    const size_t e = (size_t)off + (size_t)ix * pstr;
    v.a = cache[e];
    if constexpr (!XZ) v.x = xrow[e];
    v.b = brow[e];
    return v;
  };
  auto cvt = [&](CR v) -> T {
    if constexpr (CK == 2)
      return (T)from_bf16(v);
    else
      return v;
  };

  // coarse ring: lane l < CSLAB owns slab point (cy0 + l / CZN, cz0 + l % CZN)
  const int nc = (n - 1) / 2 + 1;
  const int cLP = lay_pitch(nc), cLO = lay_off(nc);
  const T* __restrict__ crow = xc + (size_t)row * (size_t)lay_row(nc);
  const int cy0 = (y0 - 3) >> 1, cz0 = (z0 - 3) >> 1;
  bool cld = false;
  size_t coff = 0;
  if (tid < CSLAB) {
    const int gy = cy0 + tid / CZN, gz = cz0 + tid % CZN;
    cld = gy >= 0 && gz >= 0 && gy <= nc - 1 && gz <= nc - 1;
    if (cld) coff = (size_t)gy * cLP + gz + cLO;
  }
  auto cload = [&](int J) -> T {
    return (cld && J >= 0 && J <= nc - 1) ? crow[(size_t)J * nc * cLP + coff] : T(0);
  };
  auto cstore = [&](int J, T v) {
    if (tid < CSLAB) scs[(J & 3) * CSLAB + tid] = v;
  };
  ProlongLds<T> pco, pcs;
  // prolonged correction of plane ix of a column (zero on the boundary,
  // where every contributing coarse vertex is a boundary vertex)
  auto corr = [&](ProlongLds<T>& pc, int ix) -> T { return pc.at(scs, CSLAB, ix); };

  const int x0 = 1 + xcix * g.t.xchunk;
  const int x1 = min(x0 + g.t.xchunk, n - 1);
  const int ixs = x0 - 2;  // first plane whose y a column forms
  int chi = (x0 + 1) >> 1; // highest coarse plane stored
  for (int J = ixs >> 1; J <= chi; ++J) cstore(J, cload(J));
  T cnext = cload(chi + 1);
  __syncthreads();
  pco.init(scs, CSLAB, CZN, cy0, cz0, oy, oz, ixs);
  if (s_on) pcs.init(scs, CSLAB, CZN, cy0, cz0, sy, sz, ixs);

  // On entry to step q: y and 1/a at q-1, q, q+1 and b at q, q+1 for the
  // patch column (o*) and the slot (s*; two-point ring slots and corners use
  // plane q only)
  // Faces.  A face is shared by its two vertices: every position forms the
  // faces to +y and +z of plane p once into LDS (from 1/a of plane p, stored
  // one step ahead), and every stencil column forms the face to +x of its
  // plane and keeps the one to -x from the plane before.  Faces of the last
  // row and column of the patch-with-rings are never read and not formed.
  T* __restrict__ sa = sb[0];
  auto faces_yz = [&](int p, int idx) {
    if constexpr (SHARE) {
      const int r = idx / PZ, cc = idx - (idx / PZ) * PZ;
      if (r < TY + 3) fy[p % 3][idx] = sface(sa[idx], sa[idx + PZ]);
      if (cc < TZ + 3) fz[p % 3][idx] = sface(sa[idx], sa[idx + 1]);
    }
  };

  // On entry to step q: y at q-1, q, q+1, 1/a at q, q+1, b at q, q+1 and the
  // face to +x of plane q-1 for the patch column (o*) and the slot (s*;
  // two-point ring slots and corners use plane q only)
  T oym, oyc, oyp, obm, obc, obp, orc, orp, ofb;
  T sym = T(0), syc = T(0), syp = T(0), sbm = T(1), sbc = T(1), sbp = T(1), src = T(0), srp = T(0),
    sfb = T(0);
  {
    const Raw m = load(ixs, ooff), c = load(ixs + 1, ooff),
              p = load(ixs + 2, ooff);
    oym = m.x + corr(pco, ixs);
    oyc = c.x + corr(pco, ixs + 1);
    oyp = p.x + corr(pco, ixs + 2);
    obm = cvt(m.a); obc = cvt(c.a); obp = cvt(p.a);
    ofb = sface(obm, obc);
    orc = c.b; orp = p.b;
    if (SHARE) sa[oidx] = obc;
    if (s_on) {
      const Raw sm = load(ixs, soff), sc = load(ixs + 1, soff),
                sp = load(ixs + 2, soff);
      sym = sm.x + corr(pcs, ixs);
      syc = sc.x + corr(pcs, ixs + 1);
      syp = sp.x + corr(pcs, ixs + 2);
      sbm = cvt(sm.a); sbc = cvt(sc.a); sbp = cvt(sp.a);
      sfb = sface(sbm, sbc);
      src = sc.b; srp = sp.b;
      if (SHARE) sa[sidx] = sbc;
    }
  }
  if (SHARE) {
    __syncthreads();
    faces_yz(ixs + 1, oidx);
    if (s_on) faces_yz(ixs + 1, sidx);
    __syncthreads();
  }

  // patch column: x3 at q-2, q-1, b at q-1, 1/a and the face to +x of plane
  // q-2, and the reciprocal diagonal of plane q-1 (formed by the x3 step
  // there, from the faces and in the order the x4 step would use)
  T x3a = T(0), x3b = T(0), rm_ = T(0), ofa = T(0), obmm = T(1), odb = T(0);
  double dot = 0.0;

  for (int q = x0 - 1; q <= x1; ++q) {
    const Raw on = load(q + 2, ooff);
    Raw sn{T(0), T(0), one};
    if (s_on) sn = load(q + 2, soff);
    if (((q + 3) >> 1) > chi) {
      ++chi;
      cstore(chi, cnext);
      cnext = cload(chi + 1);
    }

    T* __restrict__ b3 = sb[SHARE ? 0 : q % 3];  // 1/a of plane q (without SHARE)
    s1[oidx] = oyc;
    b3[oidx] = SHARE ? obp : obc;
    if (s_on) {
      s1[sidx] = syc;
      b3[sidx] = SHARE ? sbp : sbc;
    }
    __syncthreads();
    const T ocn = corr(pco, q + 2);
    const T scn = s_on ? corr(pcs, q + 2) : T(0);
    faces_yz(q + 1, oidx);
    if (s_on) faces_yz(q + 1, sidx);

    // x3 on plane q: patch and one-point ring
    const bool qin = q >= 1 && q <= n - 2;
    const T* __restrict__ fyq = fy[SHARE ? q % 3 : 0];
    const T* __restrict__ fzq = fz[SHARE ? q % 3 : 0];
    // faces to -y, +y, -z, +z of LDS position idx (centre 1/a bv) on plane q
    auto yz4 = [&](int idx, T bv, T& fym, T& fyp, T& fzm, T& fzp) {
      if constexpr (SHARE) {
        fym = fyq[idx - PZ]; fyp = fyq[idx]; fzm = fzq[idx - 1]; fzp = fzq[idx];
      } else {
        fym = sface(bv, b3[idx - PZ]); fyp = sface(bv, b3[idx + PZ]);
        fzm = sface(bv, b3[idx - 1]); fzp = sface(bv, b3[idx + 1]);
      }
    };
    const T ofc = sface(obc, obp);
    T x3c = T(0), odc = T(0);
    if (qin && o_int) {
      const T fxm = ofb, fxp = ofc;
      T fym, fyp, fzm, fzp;
      yz4(oidx, obc, fym, fyp, fzm, fzp);
      const T diag = ((fxm + fxp) + (fym + fyp)) + (fzm + fzp);
      const T off = ((fxm * oym + fxp * oyp) + (fym * s1[oidx - PZ] + fyp * s1[oidx + PZ])) +
                    (fzm * s1[oidx - 1] + fzp * s1[oidx + 1]);
      odc = srcp(ih2 * diag);
      x3c = oyc + omega_a * (orc - ih2 * (diag * oyc - off)) * odc;
    }
    T* __restrict__ x3s = s3[q & 1];
    x3s[oidx] = x3c;
    const T sfc = sface(sbc, sbp);
    if (ring1) {
      T v = T(0);
      if (qin && s_int) {
        const T hxm = sfb, hxp = sfc;
        T hym, hyp, hzm, hzp;
        yz4(sidx, sbc, hym, hyp, hzm, hzp);
        const T hd = ((hxm + hxp) + (hym + hyp)) + (hzm + hzp);
        const T hoff = ((hxm * sym + hxp * syp) + (hym * s1[sidx - PZ] + hyp * s1[sidx + PZ])) +
                       (hzm * s1[sidx - 1] + hzp * s1[sidx + 1]);
        v = syc + omega_a * (src - ih2 * (hd * syc - hoff)) * srcp(ih2 * hd);
      }
      x3s[sidx] = v;
    }
    __syncthreads();

    // x4 on plane q-1 from x3 of planes q-2, q-1 (LDS with ring), q and the
    // faces of plane q-1
    const int qr = q - 1;
    if (qr >= x0 && o_int) {
      const T* __restrict__ x3p = s3[qr & 1];
      const T fxm = ofa, fxp = ofb;
      T fym, fyp, fzm, fzp;
      if constexpr (SHARE) {
        const T* __restrict__ fyr = fy[qr % 3];
        const T* __restrict__ fzr = fz[qr % 3];
        fym = fyr[oidx - PZ]; fyp = fyr[oidx]; fzm = fzr[oidx - 1]; fzp = fzr[oidx];
      } else {
        const T* __restrict__ bq = sb[qr % 3];
        fym = sface(obm, bq[oidx - PZ]); fyp = sface(obm, bq[oidx + PZ]);
        fzm = sface(obm, bq[oidx - 1]); fzp = sface(obm, bq[oidx + 1]);
      }
      const T diag = ((fxm + fxp) + (fym + fyp)) + (fzm + fzp);
      const T off = ((fxm * x3a + fxp * x3c) + (fym * x3p[oidx - PZ] + fyp * x3p[oidx + PZ])) +
                    (fzm * x3p[oidx - 1] + fzp * x3p[oidx + 1]);
      // FP64: odb is srcp(ih2 * diag) of this column and plane as the x3
      // step formed it (a three-operation reciprocal); FP32 forms it again
      // (one instruction, and the kept value would cost occupancy)
      const T dinv = sizeof(T) == 8 ? odb : srcp(ih2 * diag);
      const T val = x3b + omega_b * (rm_ - ih2 * (diag * x3b - off)) * dinv;
      const size_t e = base + ((size_t)qr * n + oy) * LP + oz + LO;
      __builtin_nontemporal_store(val, &xout[e]);
      if (partial) dot += (double)rm_ * (double)val;
    }

    // advance one plane
    x3a = x3b;
    x3b = x3c;
    odb = odc;
    rm_ = orc;
    ofa = ofb; ofb = ofc;
    obmm = obm;
    oym = oyc; oyc = oyp; oyp = on.x + ocn;
    obm = obc; obc = obp; obp = cvt(on.a);
    orc = orp; orp = on.b;
    if (s_on) {
      sfb = sfc;
      sym = syc; syc = syp; syp = sn.x + scn;
      sbm = sbc; sbc = sbp; sbp = cvt(sn.a);
      src = srp; srp = sn.b;
    }
  }
  if (partial != nullptr && prob >= top_begin) {
    const double s = block_sum<NT>(dot, sred);
    if (threadIdx.x == 0) partial[poff[prob] + tile] = s;
  }
}

// ---------------------------------------------------------------------------
// Vector form of the two fused smoothing passes (k_pre2v, k_post2v), for grids
// of 11 and more vertices whose z line is at most 64 vectors of 16 bytes long.
//
// What bounds it: memory latency and LDS, not arithmetic.  The scalar form
// (k_pre2r, k_post2: one point per lane on an 8 x 64 patch, y and z neighbours
// through LDS) issued about 220 VALU and 40 LDS instructions per 64 points and
// reached 3.0-3.4 TB/s of the bytes it needs in FP64 and 2.1-2.6 in FP32.  Here
// a lane owns V = 2 (FP64) or 4 (FP32) consecutive z points of one row: loads
// and stores are 16 bytes a lane, half or three quarters of the z neighbours
// are the lane's own, and a workgroup holds whole z lines, so the rings exist
// in y alone.  On the 129^3 rows a wave's plane step issues 162 VALU and 12 LDS
// instructions (pre-smoothing) or 169 and 17 (post-smoothing) per 128 points in
// FP64, 220 and 13 or 240 and 23 per 256 in FP32; the VALU is busy 0.4-0.5 of
// the time, and waves wait for memory or LDS half of theirs.  One barrier a plane:
// the planes in LDS are double buffered.
//
// A workgroup forms the middle stage on R rows (thread = row x lane) and the
// output on the R - 2 inner ones; the first and last row's threads also load
// the row beyond theirs.  Where a grid's whole plane fits 512 threads the tile
// covers it (full) and nothing is formed twice.  Otherwise R is what fills 256
// threads (three workgroups per CU at 150 VGPRs), and 10 for lines of more than
// 32 vectors, whose chunk then spans the whole line if that still gives every
// CU a workgroup (make_vtile).
//
// The harmonic faces are formed without their factor 2, which the scale 2 h^-2
// takes over, and a step is x + omega (D^-1 (b / (2 h^-2) + sum of faces times
// neighbours) - x): the scalar passes' steps up to rounding.
//
// Measured on synthetic rows, scalar against vector form, microseconds a pass
// (post-smoothing / pre-smoothing): FP64 16 x 129^3 355/371 -> 272/258,
// 96 x 65^3 264/256 -> 219/221, 416 x 33^3 161/142 -> 121/128, 1696 x 17^3
// 76/56 -> 59/59; FP32 211/187 -> 146/146, 156/132 -> 111/111, 95/63 -> 51/51,
// 49/33 -> 32/30, 4 x 257^3 415/388 -> 277/264, 70 x 49^3 90/66 -> 39/36; FP32
// with the bfloat16 cache 266/248 -> 170/170 (129^3), 190/155 -> 131/115 (65^3).
// Whole estimates 9^3..129^3: FP64 63.2 -> 58.5 ms, FP32 cycles 52.2 -> 48.1,
// bfloat16 cache 62.3 -> 55.4; 9^3..257^3 with FP32 cycles 160 -> 147.
// ---------------------------------------------------------------------------
template <typename T>
struct VecOf {
  static constexpr int V = 16 / (int)sizeof(T);
  typedef T type __attribute__((ext_vector_type(16 / sizeof(T))));
  typedef type utype __attribute__((aligned(sizeof(T))));   // as it lies in memory
};

VTile make_vtile(int n, int elem, int tile_y, int xchunk, int rows) {
  VTile v{};
  const int V = 16 / elem, m = n - 2;
  xchunk = chunk_planes(xchunk);
  // lines that are no whole number of vectors (11 and 15 vertices in FP32) or
  // longer than 64 of them, 9^3 and below (k_vsmall) and the 4 x 64 tiles
  // (which keep the separate passes) have no vector form
  if (m <= 8 || (n - 1) % V || (n - 1) / V > 64 || (m > 32 && tile_y == 4)) return v;
  v.LZ = (n - 1) / V;
  v.full = m * v.LZ <= 512;
  v.R = v.full ? m : v.LZ > 32 ? 10 : (256 / v.LZ) & ~1;
  v.nty = v.full ? 1 : cdiv(m, v.R - 2);
  v.PZ = V * (v.LZ + 1);
  v.cyn = v.R / 2 + 3;
  v.czn = (n - 1) / 2 + 1;
  const int threads = v.R * v.LZ;
  // y, 1/a and the middle stage of two planes; the coarse ring or (full tiles)
  // the x-restricted plane
  v.lds = (6 * (v.R + 2) * v.PZ + std::max(4 * v.cyn * v.czn, (v.R + 2) * v.PZ) + V) * elem;
  // The chunk: the least of split_chunk's cost (without its 15% threshold), over
  // halves of the given length and also longer ones, up to the whole line.  Odd
  // chunk lengths stay as given (the x-restricted residual needs even ones).
  int best = m <= xchunk ? m : xchunk;
  if (rows > 0 && (m <= xchunk || xchunk % 2 == 0)) {
    const long long fit = 256LL * max(1, 12 / cdiv(threads, 64));
    auto cost = [&](int ch) {
      const long long wg = (long long)rows * v.nty * cdiv(m, ch);
      return ((wg + fit - 1) / fit) * (ch + 6);
    };
    int ch = m + (m & 1);
    if (xchunk < m)
      for (ch = xchunk; 2 * ch < m; ch *= 2) {}
    best = m;
    for (;; ch /= 2) {
      if (ch < m && cost(ch) < cost(best)) best = ch;
      if (ch % 4) break;
    }
  }
  v.xchunk = best;
  v.tiles = v.nty * cdiv(m, best);
  return v;
}

// Geometry of one workgroup of the vector passes and its loads.  A value of
// plane ix is addressed by a scalar base and the lane's 32-bit byte offset;
// rows and planes beyond the grid read the nearest one inside (their values
// only reach results that are set to zero or discarded).
template <typename T, int CK>
struct VGeo {
  static constexpr int V = VecOf<T>::V;
  using VT = typename VecOf<T>::type;
  using VU = typename VecOf<T>::utype;
  static constexpr uint32_t CS = CK == 2 ? 2 : sizeof(T);   // bytes of a cached coefficient
  int n, tile, prob, r, l, j, jb, js;
  int x0, x1, o, so, rows2;   // LDS: own and secondary slot, elements of one plane of R + 2 rows
  bool rint, out, edge, first, s_on, idle;
  size_t base;
  uint32_t pstr, eo, es;      // plane stride, element offsets of the own and the secondary row
  const char* cache;
  __device__ int clampj(int a) const { return min(max(a, 0), n - 1); }
  __device__ void init(const GridArgs& g) {
    n = g.n;
    const int LP = lay_pitch(n), LO = lay_off(n);
    const int bid = xcd_swizzle(blockIdx.x, gridDim.x);
    const int row = bid / g.v.tiles;
    tile = bid - row * g.v.tiles;
    prob = g.row0 + row;
    idle = g.scal && !g.scal[prob].active;   // uniform
    const int ty = tile % g.v.nty, xc = tile / g.v.nty;
    r = threadIdx.x / g.v.LZ;
    l = threadIdx.x - r * g.v.LZ;
    jb = g.v.full ? 1 : ty * (g.v.R - 2);
    j = jb + r;
    rint = j >= 1 && j <= n - 2;
    out = rint && (g.v.full || (r >= 1 && r <= g.v.R - 2));
    edge = l == g.v.LZ - 1;
    first = l == 0;
    s_on = r == 0 || r == g.v.R - 1;
    js = r == 0 ? j - 1 : j + 1;
    rows2 = (g.v.R + 2) * g.v.PZ;
    o = (r + 1) * g.v.PZ + V * (l + 1);
    so = (r == 0 ? 0 : g.v.R + 1) * g.v.PZ + V * (l + 1);
    base = (size_t)row * (size_t)g.stride;
    pstr = (uint32_t)n * (uint32_t)LP;
    eo = (uint32_t)(clampj(j) * LP + 1 + V * l + LO);
    es = (uint32_t)(clampj(js) * LP + 1 + V * l + LO);
    cache = (const char*)g.cache + (size_t)prob * (size_t)g.stride * CS;
    x0 = 1 + xc * g.v.xchunk;
    x1 = min(x0 + g.v.xchunk, n - 1);
  }
  __device__ size_t plane(int ix) const { return (size_t)clampj(ix) * pstr; }   // uniform
  __device__ VT load(const T* p, int ix, uint32_t e) const {
    return *(const VU*)((const char*)(p + plane(ix)) + e * (uint32_t)sizeof(T));
  }
  __device__ void store(T* p, int ix, const VT& v) const {
    __builtin_nontemporal_store(v, (VU*)((char*)(p + base + (size_t)ix * pstr) + eo * (uint32_t)sizeof(T)));
  }
  __device__ VT load_a(int ix, uint32_t e) const {   // 1/a
    const char* p = cache + plane(ix) * CS + e * CS;
    if constexpr (CK == 2) {
      typedef uint16_t u16x4 __attribute__((ext_vector_type(4), aligned(2)));
      const u16x4 h = *(const u16x4*)p;
      VT v;
#pragma unroll
      for (int k = 0; k < 4; ++k) v[k] = from_bf16(h[k]);
      return v;
    } else {
      return *(const VU*)p;
    }
  }
  __device__ T load_a0(int ix) const {   // 1/a at z = 0, left of the row's first vector
    const char* p = cache + plane(ix) * CS + (eo - 1) * CS;
    if constexpr (CK == 2)
      return (T)from_bf16(*(const uint16_t*)p);
    else
      return *(const T*)p;
  }
  __device__ static VT fill(T a) {
    VT v;
#pragma unroll
    for (int e = 0; e < V; ++e) v[e] = a;
    return v;
  }
  // half the harmonic faces between two vectors of 1/a
  __device__ static VT face2(const VT& a, const VT& b) {
    VT v;
#pragma unroll
    for (int e = 0; e < V; ++e) v[e] = srcp((T)(a[e] + b[e]));
    return v;
  }
};

// half faces of a row's vector to its z neighbours (a: the row in LDS at o)
template <typename T, typename VT>
__device__ __forceinline__ void zfaces(const T* a, int o, const VT& ac, T (&fz)[VecOf<T>::V + 1]) {
  constexpr int V = VecOf<T>::V;
  fz[0] = srcp((T)(a[o - 1] + ac[0]));
#pragma unroll
  for (int e = 1; e < V; ++e) fz[e] = srcp((T)(ac[e - 1] + ac[e]));
  fz[V] = srcp((T)(ac[V - 1] + a[o + V]));
}
// of + the y and z terms of the stencil at row slot o of t (own values v)
template <typename T, typename VT>
__device__ __forceinline__ VT yz_terms(VT of, const T* t, int o, int PZ, const VT& v, const VT& fym,
                                       const VT& fyp, const T (&fz)[VecOf<T>::V + 1]) {
  constexpr int V = VecOf<T>::V;
  const VT tym = *(const VT*)(t + o - PZ), typ = *(const VT*)(t + o + PZ);
  const T tl = t[o - 1], tr = t[o + V];
#pragma unroll
  for (int e = 0; e < V; ++e) {
    T s = of[e];
    s += fym[e] * tym[e];
    s += fyp[e] * typ[e];
    s += fz[e] * (e > 0 ? v[e > 0 ? e - 1 : 0] : tl);
    s += fz[e + 1] * (e < V - 1 ? v[e < V - 1 ? e + 1 : 0] : tr);
    of[e] = s;
  }
  return of;
}

// Zero column z = 0 of the two value arrays and the rows beyond the tile of the
// second one (read by discarded rows only).
template <typename T, int CK>
__device__ __forceinline__ void vec_lds_init(const VGeo<T, CK>& G, T* sy, T* s3) {
  if (G.first) {
#pragma unroll
    for (int b = 0; b < 2; ++b) {
      sy[b * G.rows2 + G.o - 1] = T(0);
      s3[b * G.rows2 + G.o - 1] = T(0);
    }
  }
  if (G.s_on) {
#pragma unroll
    for (int b = 0; b < 2; ++b)
      *(typename VecOf<T>::type*)(s3 + b * G.rows2 + G.so) = VGeo<T, CK>::fill(T(0));
  }
}

constexpr int VEC_THREADS = 640;   // most threads of a tile (R = 10, 64 vectors)

// What the pre-smoothing pass writes beside its result: the residual, the
// residual restricted along x, or (tiles that cover the plane) the coarse grid's
// right-hand side, y and z restricted through LDS one step later.  That spares a
// launch and a round trip of h per grid and cycle: one adjoint solve on a 33^3
// grid (both states) 1.77 -> 1.67 ms, an objective on 65^3 3.31 -> 3.23 ms
enum PreOut { PR_RESID = 0, PR_HALF = 1, PR_COARSE = 2 };

// Two Chebyshev steps from x = 0 and the residual (k_pre2r's pass).  In step q
// the middle stage x2 of plane q and the residual of plane q - 1 are formed;
// planes q + 2 of b, 1/D and 1/a load meanwhile.
template <typename T, int CK, int OUT>
__global__ void __launch_bounds__(VEC_THREADS)
    k_pre2v(GridArgs g, const T* __restrict__ dinv, const T* __restrict__ rhs,
            T* __restrict__ xout, T* __restrict__ rout, T omega1, T omega2) {
  constexpr bool RH = OUT != PR_RESID;
  using Geo = VGeo<T, CK>;
  using VT = typename Geo::VT;
  constexpr int V = Geo::V;
  extern __shared__ __align__(16) unsigned char smem[];
  Geo G;
  G.init(g);
  if (G.idle) return;
  const int n = G.n, PZ = g.v.PZ, o = G.o, x0 = G.x0, x1 = G.x1;
  T* const sy = (T*)smem;            // x1 of planes q and q - 1
  T* const sa = sy + 2 * G.rows2;    // 1/a
  T* const s3 = sa + 2 * G.rows2;    // x2 of planes q - 1 and q - 2
  T* const sh = s3 + 2 * G.rows2;    // PR_COARSE: the last x-restricted plane
  vec_lds_init(G, sy, s3);
  // coarse plane I from sh (row j of the grid in LDS row j, the tile being full)
  const int nc = (n - 1) / 2 + 1, mc = nc - 2;
  auto coarse = [&](int I) {
    T* __restrict__ c = rout + (size_t)(G.base / (size_t)g.stride) * (size_t)lay_row(nc) +
                        (size_t)I * nc * lay_pitch(nc) + lay_off(nc);
    for (int i = threadIdx.x; i < mc * mc; i += g.v.R * g.v.LZ) {
      const int J = 1 + i / mc, K = 1 + i % mc;
      const T* p = sh + 2 * J * PZ + V - 1 + 2 * K;
      T acc = T(0);
#pragma unroll
      for (int dy = -1; dy <= 1; ++dy) {
        const T* h = p + dy * PZ;
        acc += (dy == 0 ? T(0.5) : T(0.25)) * (T(0.25) * h[-1] + T(0.5) * h[0] + T(0.25) * h[1]);
      }
      c[J * lay_pitch(nc) + K] = acc;
    }
  };
  int pend = 0;   // coarse plane in sh not yet written out (0: none)
  const T* __restrict__ brow = rhs + G.base;
  const T* __restrict__ drow = dinv + G.base;
  const VT zero = Geo::fill(T(0));
  const int qend = RH ? min(x1 + 1, n - 1) : x1;
  const T i2 = T(2) * (T)g.ih2, kk = T(1) / i2;
  // state on entry to step q: x1 and 1/a of planes q and q + 1, b of both, the
  // b and x- terms of x2 on plane q (S1) and of the residual on q - 1 (S2), x2
  // of plane q - 1 with its y and z faces and diagonal, the face q - 1 | q
  VT yc, yn, S1, fxm, ac, an, bc, bn;
  VT S2 = zero, x2p = zero, dg2 = zero, fym2 = zero, fyp2 = zero, hacc = zero;
  T fz2[V + 1];
#pragma unroll
  for (int e = 0; e <= V; ++e) fz2[e] = T(0);
  VT sys = zero, sas = Geo::fill(T(1));
  T a0c = T(1);
  {
    const int q = x0 - 1;
    const VT am = G.load_a(q - 1, G.eo);
    ac = G.load_a(q, G.eo);
    an = G.load_a(q + 1, G.eo);
    const VT ym = (omega1 * G.load(brow, q - 1, G.eo)) * G.load(drow, q - 1, G.eo);
    bc = G.load(brow, q, G.eo);
    yc = (omega1 * bc) * G.load(drow, q, G.eo);
    bn = G.load(brow, q + 1, G.eo);
    yn = (omega1 * bn) * G.load(drow, q + 1, G.eo);
    if (G.first) a0c = G.load_a0(q);
    fxm = Geo::face2(am, ac);
    S1 = kk * bc + (q >= 1 ? fxm * ym : zero);
    if (G.s_on) {
      sys = (omega1 * G.load(brow, q, G.es)) * G.load(drow, q, G.es);
      sas = G.load_a(q, G.es);
    }
  }

  for (int q = x0 - 1; q <= qend; ++q) {
    const VT rb = G.load(brow, q + 2, G.eo);
    const VT rd = G.load(drow, q + 2, G.eo);
    const VT ra = G.load_a(q + 2, G.eo);
    T ra0 = T(1);
    if (G.first) ra0 = G.load_a0(q + 1);
    VT rsb = zero, rsd = zero, rsa = zero;
    if (G.s_on) {
      rsb = G.load(brow, q + 1, G.es);
      rsd = G.load(drow, q + 1, G.es);
      rsa = G.load_a(q + 1, G.es);
    }
    T* const y_ = sy + (q & 1) * G.rows2;
    T* const a_ = sa + (q & 1) * G.rows2;
    T* const t_ = s3 + (q & 1) * G.rows2;
    *(VT*)(y_ + o) = yc;
    *(VT*)(a_ + o) = ac;
    *(VT*)(t_ + o) = x2p;
    if (G.first) a_[o - 1] = a0c;
    if (G.s_on) {
      *(VT*)(y_ + G.so) = sys;
      *(VT*)(a_ + G.so) = sas;
    }
    __syncthreads();
    if (OUT == PR_COARSE && pend) {   // uniform
      coarse(pend);
      pend = 0;
    }

    const VT fxp = Geo::face2(ac, an);
    const VT fym = Geo::face2(ac, *(const VT*)(a_ + o - PZ));
    const VT fyp = Geo::face2(ac, *(const VT*)(a_ + o + PZ));
    T fz[V + 1];
    zfaces<T, VT>(a_, o, ac, fz);
    const VT of = yz_terms<T, VT>(S1 + fxp * yn, y_, o, PZ, yc, fym, fyp, fz);
    VT dg, x2;
#pragma unroll
    for (int e = 0; e < V; ++e) {
      dg[e] = ((fxm[e] + fxp[e]) + (fym[e] + fyp[e])) + (fz[e] + fz[e + 1]);
      x2[e] = yc[e] + omega2 * (of[e] * srcp(dg[e]) - yc[e]);
    }
    if (!(q >= 1 && q <= n - 2 && G.rint)) x2 = zero;
    if (G.edge) x2[V - 1] = T(0);   // z = n - 1

    const int qr = q - 1;
    if (qr >= x0 && G.out) {
      const VT o2 = yz_terms<T, VT>(S2 + fxm * x2, t_, o, PZ, x2p, fym2, fyp2, fz2);
      VT rv = i2 * (o2 - dg2 * x2p);
      if (G.edge) rv[V - 1] = T(0);
      if constexpr (RH) {
        if (qr < x1) G.store(xout, qr, x2p);
        if (qr & 1) {
          // r(qr) closes coarse plane (qr - 1) / 2 and opens (qr + 1) / 2
          if (qr >= x0 + 2) {
            const VT h = hacc + T(0.25) * rv;
            if constexpr (OUT == PR_COARSE)
              *(VT*)(sh + o) = h;
            else
              G.store(rout, (qr - 1) >> 1, h);
          }
          hacc = T(0.25) * rv;
        } else {
          hacc = hacc + T(0.5) * rv;
        }
      } else {
        G.store(xout, qr, x2p);
        G.store(rout, qr, rv);
      }
    }
    if (OUT == PR_COARSE && (qr & 1) && qr >= x0 + 2) pend = (qr - 1) >> 1;

    S2 = kk * bc + fxm * x2p;
    S1 = kk * bn + fxp * yc;
    bc = bn;
    bn = rb;
    fym2 = fym; fyp2 = fyp; dg2 = dg; x2p = x2;
#pragma unroll
    for (int e = 0; e <= V; ++e) fz2[e] = fz[e];
    fxm = fxp;
    ac = an;
    an = ra;
    yc = yn;
    yn = (omega1 * rb) * rd;
    a0c = ra0;
    if (G.s_on) {
      sys = (omega1 * rsb) * rsd;
      sas = rsa;
    }
  }
  if (OUT == PR_COARSE && pend) {
    __syncthreads();
    coarse(pend);
  }
}

// Two Chebyshev steps after the coarse-grid correction (k_post2's pass; XZ: from
// x = 0).  In step q the first step x3 of plane q and the second x4 of plane
// q - 1 are formed.  The coarse planes of the tile's footprint sit in a
// four-plane LDS ring; a row forms its correction of plane q + 2 from it.
template <typename T, int CK, bool XZ>
__global__ void __launch_bounds__(VEC_THREADS)
    k_post2v(GridArgs g, const T* __restrict__ xin, const T* __restrict__ xc,
             const T* __restrict__ rhs, T* __restrict__ xout, const int* __restrict__ poff,
             double* __restrict__ partial, int top_begin, T omega_a, T omega_b) {
  using Geo = VGeo<T, CK>;
  using VT = typename Geo::VT;
  constexpr int V = Geo::V;
  extern __shared__ __align__(16) unsigned char smem[];
  __shared__ double sred[VEC_THREADS / 64];
  Geo G;
  G.init(g);
  if (G.idle) return;
  const int n = G.n, PZ = g.v.PZ, o = G.o, x0 = G.x0, x1 = G.x1;
  const int tid = threadIdx.x, NT = g.v.R * g.v.LZ;
  T* const sy = (T*)smem;            // y of planes q and q - 1
  T* const sa = sy + 2 * G.rows2;    // 1/a
  T* const s3 = sa + 2 * G.rows2;    // x3 of planes q - 1 and q - 2
  T* const scs = s3 + 2 * G.rows2;   // coarse plane J in slot J & 3
  const T* __restrict__ xrow = XZ ? nullptr : xin + G.base;
  const T* __restrict__ brow = rhs + G.base;
  const VT zero = Geo::fill(T(0));
  auto ldx = [&](int ix, uint32_t e) -> VT {
    if constexpr (XZ)
      return zero;
    else
      return G.load(xrow, ix, e);
  };

  // coarse ring: cyn rows from cy0 by the whole coarse line; a thread stages
  // slots tid and tid + NT
  const int nc = (n - 1) / 2 + 1, czn = g.v.czn, slab = g.v.cyn * czn;
  const int cLP = lay_pitch(nc), cLO = lay_off(nc);
  const T* __restrict__ crow = xc + (size_t)(G.base / (size_t)g.stride) * (size_t)lay_row(nc);
  const int cy0 = max(G.jb - 1, 0) >> 1;
  const size_t cpl = (size_t)nc * cLP;
  auto slot = [&](int i, uint32_t& e) -> bool {
    const int a = i / czn;
    e = (uint32_t)((cy0 + a) * cLP + (i - a * czn) + cLO);
    return i < slab && cy0 + a <= nc - 1;
  };
  uint32_t co0, co1;
  const bool c0 = slot(tid, co0), c1 = slot(tid + NT, co1);
  auto cload = [&](bool on, uint32_t e, int J) -> T {
    return (on && J >= 0 && J <= nc - 1) ? crow[(size_t)J * cpl + e] : T(0);
  };
  auto cstore = [&](int J, T a, T b) {
    T* s = scs + (J & 3) * slab;
    if (tid < slab) s[tid] = a;
    if (tid + NT < slab) s[tid + NT] = b;
  };
  // y-interpolated values of coarse plane J under a row, then the trilinear
  // correction of its V points on plane ix
  struct Line {
    T w[V / 2 + 1];
  };
  auto line = [&](int J, int lc, int dy) -> Line {
    const T* p = scs + (J & 3) * slab + lc;
    Line c;
#pragma unroll
    for (int k = 0; k <= V / 2; ++k) c.w[k] = T(0.5) * (p[k] + p[k + dy]);
    return c;
  };
  auto corr = [&](int ix, int lc, int dy) -> VT {
    Line c = line(ix >> 1, lc, dy);
    if (ix & 1) {   // uniform
      const Line d = line((ix >> 1) + 1, lc, dy);
#pragma unroll
      for (int k = 0; k <= V / 2; ++k) c.w[k] = T(0.5) * (c.w[k] + d.w[k]);
    }
    VT y;
#pragma unroll
    for (int e = 0; e < V; e += 2) {
      y[e] = T(0.5) * (c.w[e / 2] + c.w[e / 2 + 1]);
      y[e + 1] = c.w[e / 2 + 1];
    }
    return y;
  };
  const int jc = G.clampj(G.j), jsc = G.clampj(G.js);
  const int lcp = ((jc >> 1) - cy0) * czn + (V / 2) * G.l, dyp = (jc & 1) ? czn : 0;
  const int lcs = ((jsc >> 1) - cy0) * czn + (V / 2) * G.l, dys = (jsc & 1) ? czn : 0;

  const int ixs = x0 - 2;    // first plane whose y a row forms
  int chi = (x0 + 1) >> 1;   // highest coarse plane stored
  for (int J = ixs >> 1; J <= chi; ++J) cstore(J, cload(c0, co0, J), cload(c1, co1, J));
  T cn0 = cload(c0, co0, chi + 1), cn1 = cload(c1, co1, chi + 1);
  vec_lds_init(G, sy, s3);
  __syncthreads();

  const T kk = T(1) / (T(2) * (T)g.ih2);
  // state on entry to step q: y and 1/a of planes q and q + 1, b of q - 1 and
  // q, the b and x- terms of x3 on plane q (S1) and of x4 on q - 1 (S2), x3 of
  // plane q - 1 with its y and z faces and reciprocal diagonal, the face
  // q - 1 | q
  VT yc, yn, S1, fxm, ac, an, bc;
  VT bm = zero, S2 = zero, x3p = zero, rd2 = zero, fym2 = zero, fyp2 = zero;
  T fz2[V + 1];
#pragma unroll
  for (int e = 0; e <= V; ++e) fz2[e] = T(0);
  VT sys = zero, sas = Geo::fill(T(1));
  T a0c = T(1);
  {
    const VT am = G.load_a(ixs, G.eo);
    ac = G.load_a(ixs + 1, G.eo);
    an = G.load_a(ixs + 2, G.eo);
    const VT ym = ldx(ixs, G.eo) + corr(ixs, lcp, dyp);
    yc = ldx(ixs + 1, G.eo) + corr(ixs + 1, lcp, dyp);
    yn = ldx(ixs + 2, G.eo) + corr(ixs + 2, lcp, dyp);
    bc = G.load(brow, ixs + 1, G.eo);
    if (G.first) a0c = G.load_a0(ixs + 1);
    fxm = Geo::face2(am, ac);
    S1 = kk * bc + (ixs >= 0 ? fxm * ym : zero);
    if (G.s_on) {
      sys = ldx(ixs + 1, G.es) + corr(ixs + 1, lcs, dys);
      sas = G.load_a(ixs + 1, G.es);
    }
  }
  double dot = 0.0;
  const bool want = partial != nullptr && G.prob >= top_begin;

  for (int q = x0 - 1; q <= x1; ++q) {
    const VT rx = ldx(q + 2, G.eo);
    const VT ra = G.load_a(q + 2, G.eo);
    const VT rb = G.load(brow, q + 1, G.eo);
    T ra0 = T(1);
    if (G.first) ra0 = G.load_a0(q + 1);
    VT rsx = zero, rsa = zero;
    if (G.s_on) {
      rsx = ldx(q + 1, G.es);
      rsa = G.load_a(q + 1, G.es);
    }
    if (((q + 3) >> 1) > chi) {
      ++chi;
      cstore(chi, cn0, cn1);
      cn0 = cload(c0, co0, chi + 1);
      cn1 = cload(c1, co1, chi + 1);
    }
    T* const y_ = sy + (q & 1) * G.rows2;
    T* const a_ = sa + (q & 1) * G.rows2;
    T* const t_ = s3 + (q & 1) * G.rows2;
    *(VT*)(y_ + o) = yc;
    *(VT*)(a_ + o) = ac;
    *(VT*)(t_ + o) = x3p;
    if (G.first) a_[o - 1] = a0c;
    if (G.s_on) {
      *(VT*)(y_ + G.so) = sys;
      *(VT*)(a_ + G.so) = sas;
    }
    __syncthreads();

    const VT fxp = Geo::face2(ac, an);
    const VT fym = Geo::face2(ac, *(const VT*)(a_ + o - PZ));
    const VT fyp = Geo::face2(ac, *(const VT*)(a_ + o + PZ));
    T fz[V + 1];
    zfaces<T, VT>(a_, o, ac, fz);
    const VT of = yz_terms<T, VT>(S1 + fxp * yn, y_, o, PZ, yc, fym, fyp, fz);
    VT rd, x3;
#pragma unroll
    for (int e = 0; e < V; ++e) {
      rd[e] = srcp((T)(((fxm[e] + fxp[e]) + (fym[e] + fyp[e])) + (fz[e] + fz[e + 1])));
      x3[e] = yc[e] + omega_a * (of[e] * rd[e] - yc[e]);
    }
    if (!(q >= 1 && q <= n - 2 && G.rint)) x3 = zero;
    if (G.edge) x3[V - 1] = T(0);   // z = n - 1

    if (q - 1 >= x0 && G.out) {
      const VT o2 = yz_terms<T, VT>(S2 + fxm * x3, t_, o, PZ, x3p, fym2, fyp2, fz2);
      VT v = x3p + omega_b * (o2 * rd2 - x3p);
      if (G.edge) v[V - 1] = T(0);
      G.store(xout, q - 1, v);
      if (want) {
#pragma unroll
        for (int e = 0; e < V; ++e) dot += (double)bm[e] * (double)v[e];
      }
    }

    S2 = kk * bc + fxm * x3p;
    bm = bc;
    bc = rb;
    S1 = kk * rb + fxp * yc;
    fym2 = fym; fyp2 = fyp; rd2 = rd; x3p = x3;
#pragma unroll
    for (int e = 0; e <= V; ++e) fz2[e] = fz[e];
    fxm = fxp;
    ac = an;
    an = ra;
    yc = yn;
    yn = rx + corr(q + 2, lcp, dyp);
    a0c = ra0;
    if (G.s_on) {
      sys = rsx + corr(q + 1, lcs, dys);
      sas = rsa;
    }
  }
  if (want) {
    // the last wave may be partly filled: its missing lanes add nothing
    const int lane = tid & 63, live = min(64, NT - (tid & ~63));
#pragma unroll
    for (int k = 32; k > 0; k >>= 1) {
      const double t = __shfl_down(dot, k, 64);
      if (lane + k < live) dot += t;
    }
    if (lane == 0) sred[tid >> 6] = dot;
    __syncthreads();
    if (tid == 0) {
      double s = 0.0;
      for (int w = 0; w < (NT + 63) >> 6; ++w) s += sred[w];
      partial[poff[G.prob] + G.tile] = s;
    }
  }
}

template <typename T, int CK>
static void launch_pre2v(const GridArgs& g, const T* dinv, const T* b, T* xout, T* rout,
                         double omega1, double omega2, bool half, hipStream_t s) {
  const dim3 grid(g.rows * g.v.tiles), block(g.v.R * g.v.LZ);
#define MLSGD_LAUNCH(OUT_)                                                                       \
  hipLaunchKernelGGL((k_pre2v<T, CK, OUT_>), grid, block, g.v.lds, s, g, dinv, b, xout, rout,    \
                     (T)omega1, (T)omega2)
  if (!half)
    MLSGD_LAUNCH(PR_RESID);
  else if (g.v.full)
    MLSGD_LAUNCH(PR_COARSE);
  else
    MLSGD_LAUNCH(PR_HALF);
#undef MLSGD_LAUNCH
}
template <typename T, int CK>
static void launch_post2v(const GridArgs& g, const T* xin, const T* xc, const T* b, T* xout,
                          double omega_a, double omega_b, const int* poff, double* partial,
                          int top_begin, hipStream_t s) {
  const dim3 grid(g.rows * g.v.tiles), block(g.v.R * g.v.LZ);
  if (xin)
    hipLaunchKernelGGL((k_post2v<T, CK, false>), grid, block, g.v.lds, s, g, xin, xc, b, xout, poff,
                       partial, top_begin, (T)omega_a, (T)omega_b);
  else
    hipLaunchKernelGGL((k_post2v<T, CK, true>), grid, block, g.v.lds, s, g, xin, xc, b, xout, poff,
                       partial, top_begin, (T)omega_a, (T)omega_b);
}

template <typename T>
bool march_pre2r(const GridArgs& g, const T* dinv, const T* b, T* xout, T* rout, double omega1,
                 double omega2, bool half, hipStream_t s) {
  if (!fused_tiles(g) || (half && !pre2r_half_tiles(g))) return false;
  if (g.rows <= 0) return true;
  if (g.v.R) {
    if (sizeof(T) == 4 && g.cache_bf16)
      launch_pre2v<float, 2>(g, (const float*)dinv, (const float*)b, (float*)xout, (float*)rout,
                             omega1, omega2, half, s);
    else
      launch_pre2v<T, 1>(g, dinv, b, xout, rout, omega1, omega2, half, s);
    return true;
  }
  const int nblk = g.rows * g.t.tiles_per_row;
#define MLSGD_LAUNCH(TY_, TZ_, CK_, RH_)                                                     \
  hipLaunchKernelGGL((k_pre2r<T, TY_, TZ_, CK_, RH_>), dim3(nblk), dim3(TY_ * TZ_), 0, s, g, \
                     dinv, b, xout, rout, (T)omega1, (T)omega2)
#define MLSGD_LAUNCH2(TY_, TZ_)         \
  if (b16 && half)                      \
    MLSGD_LAUNCH(TY_, TZ_, 2, true);    \
  else if (b16)                         \
    MLSGD_LAUNCH(TY_, TZ_, 2, false);   \
  else if (half)                        \
    MLSGD_LAUNCH(TY_, TZ_, 1, true);    \
  else                                  \
    MLSGD_LAUNCH(TY_, TZ_, 1, false)
  const bool b16 = sizeof(T) == 4 && g.cache_bf16;
  if (g.t.TZ == 16) {
    if constexpr (sizeof(T) == 4) {   // 11 and 15 vertices
      MLSGD_LAUNCH2(16, 16);
    }
  } else if (g.t.TY == 8) {
    MLSGD_LAUNCH2(8, 64);
  } else {
    MLSGD_LAUNCH2(16, 64);
  }
#undef MLSGD_LAUNCH2
#undef MLSGD_LAUNCH
  return true;
}
template bool march_pre2r<double>(const GridArgs&, const double*, const double*, double*,
                                  double*, double, double, bool, hipStream_t);
template bool march_pre2r<float>(const GridArgs&, const float*, const float*, float*, float*,
                                 double, double, bool, hipStream_t);

template <typename T>
bool march_post2(const GridArgs& g, const T* xin, const T* xc, const T* b, T* xout,
                 double omega_a, double omega_b, const int* poff, double* partial, int top_begin,
                 hipStream_t s) {
  if (!fused_tiles(g) || !xc) return false;
  if (g.rows <= 0) return true;
  if (g.v.R) {
    if (sizeof(T) == 4 && g.cache_bf16)
      launch_post2v<float, 2>(g, (const float*)xin, (const float*)xc, (const float*)b,
                              (float*)xout, omega_a, omega_b, poff, partial, top_begin, s);
    else
      launch_post2v<T, 1>(g, xin, xc, b, xout, omega_a, omega_b, poff, partial, top_begin, s);
    return true;
  }
  const int nblk = g.rows * g.t.tiles_per_row;
#define MLSGD_LAUNCH(TY_, TZ_, CK_, XZ_)                                                 \
  hipLaunchKernelGGL((k_post2<T, TY_, TZ_, CK_, XZ_>), dim3(nblk), dim3(TY_ * TZ_), 0, s, g, \
                     xin, xc, b, xout, poff, partial, top_begin, (T)omega_a, (T)omega_b)
#define MLSGD_LAUNCH2(TY_, TZ_)         \
  if (b16 && !xin)                      \
    MLSGD_LAUNCH(TY_, TZ_, 2, true);    \
  else if (b16)                         \
    MLSGD_LAUNCH(TY_, TZ_, 2, false);   \
  else if (!xin)                        \
    MLSGD_LAUNCH(TY_, TZ_, 1, true);    \
  else                                  \
    MLSGD_LAUNCH(TY_, TZ_, 1, false)
  const bool b16 = sizeof(T) == 4 && g.cache_bf16;
  if (g.t.TZ == 16) {
    if constexpr (sizeof(T) == 4) {   // 11 and 15 vertices
      MLSGD_LAUNCH2(16, 16);
    }
  } else if (g.t.TY == 8) {
    MLSGD_LAUNCH2(8, 64);
  } else {
    MLSGD_LAUNCH2(16, 64);
  }
#undef MLSGD_LAUNCH2
#undef MLSGD_LAUNCH
  return true;
}
template bool march_post2<double>(const GridArgs&, const double*, const double*, const double*,
                                  double*, double, double, const int*, double*, int, hipStream_t);
template bool march_post2<float>(const GridArgs&, const float*, const float*, const float*,
                                 float*, double, double, const int*, double*, int, hipStream_t);

// ---------------------------------------------------------------------------
// The V-cycle from a 9^3 grid down, 9^3 -> 5^3 -> 3^3 and back, with the
// level-by-level path's smoothing steps, transfers and exact 3^3 solve, and the
// full-multigrid start of these three grids.  One wave per problem: a chain of
// some twenty dependent steps over at most 343 points is bound by the latency of
// each step, so there is no workgroup barrier and little to recompute.  Lane
// (y, z) < 7 x 7 holds the x line of its 9^3 column in registers (right-hand
// side, iterate, faces, reciprocal diagonal), lane i < 27 one 5^3 vertex; LDS
// passes values to neighbouring lanes only, and lanes of one wave follow each
// other's LDS operations in order.  As for every grid size, row r of the 9^3, 5^3
// and 3^3 rows is problem r.  The last post-smoothing step forms <b, z> for the
// problems whose top grid is 9^3 (one partial slot per problem).
// Against one 256-thread workgroup per problem with a barrier after every step:
// 6816 problems 90 -> 60 us (FP64), one problem 11.5 -> 7.8 us; and the start of
// these grids, some 25 launches of 4 us each level by level, is one of 12 us.
// ---------------------------------------------------------------------------
__device__ __forceinline__ void wave_sync() {
  __builtin_amdgcn_fence(__ATOMIC_RELEASE, "wavefront");
  __builtin_amdgcn_wave_barrier();
  __builtin_amdgcn_fence(__ATOMIC_ACQUIRE, "wavefront");
}

constexpr int VS_WAVES = 4;   // problems per workgroup

template <typename T>
struct VsLds {          // one wave's LDS
  T v9[9 * 9 * 9];      // values (or 1/a) of the 9^3 vertices, boundary zero
  T v5[5 * 5 * 5];      // the same for 5^3
};

template <typename T, int CK>
struct VsWave {
  using CR = typename std::conditional<CK == 2, uint16_t, T>::type;
  VsLds<T>& s;
  int lane, o9, o5;            // LDS slot of plane x = 1 of the 9^3 column; of the 5^3 vertex
  bool on9, on5;
  T b[7], x[7], di[7], fx[8], fym[7], fyp[7], fzm[7], fzp[7];   // 9^3 column
  T b5, x5, di5, f5[6];                                         // 5^3 vertex (x-, x+, y-, y+, z-, z+)
  T di3;                                                        // 3^3 vertex (every lane)
  __device__ static T cvt(CR v) {
    if constexpr (CK == 2)
      return (T)from_bf16(v);
    else
      return v;
  }
  __device__ VsWave(VsLds<T>& lds, int ln) : s(lds), lane(ln) {
    const int ly = lane >> 3, lz = lane & 7;
    on9 = ly < 7 && lz < 7;
    o9 = 81 + (on9 ? (1 + ly) * 9 + 1 + lz : 10);
    on5 = lane < 27;
    const int i = on5 ? lane : 0;
    o5 = ((1 + i / 9) * 5 + 1 + (i / 3) % 3) * 5 + 1 + i % 3;
  }
  // cached 1/a of the three grids
  __device__ void load(const CR* c9, const CR* c5, const CR* c3) {
    for (int v = lane; v < 729; v += 64) s.v9[v] = cvt(c9[v]);
    for (int v = lane; v < 125; v += 64) s.v5[v] = cvt(c5[v]);
    T f3 = T(0);
    {
      const T bc = cvt(c3[13]);
      f3 = ((face(bc, cvt(c3[4])) + face(bc, cvt(c3[22]))) +
            (face(bc, cvt(c3[10])) + face(bc, cvt(c3[16])))) +
           (face(bc, cvt(c3[12])) + face(bc, cvt(c3[14])));
    }
    di3 = drcp(T(4) * f3);
    wave_sync();
  }
  // faces and reciprocal diagonals from them, then zero value arrays
  __device__ void coefficients() {
#pragma unroll
    for (int k = 0; k < 8; ++k) fx[k] = face(s.v9[o9 + (k - 1) * 81], s.v9[o9 + k * 81]);
#pragma unroll
    for (int k = 0; k < 7; ++k) {
      const int o = o9 + k * 81;
      const T bc = s.v9[o];
      fym[k] = face(bc, s.v9[o - 9]);
      fyp[k] = face(bc, s.v9[o + 9]);
      fzm[k] = face(bc, s.v9[o - 1]);
      fzp[k] = face(bc, s.v9[o + 1]);
      di[k] = drcp(T(64) * diag(k));
    }
    {
      const T bc = s.v5[o5];
      f5[0] = face(bc, s.v5[o5 - 25]);
      f5[1] = face(bc, s.v5[o5 + 25]);
      f5[2] = face(bc, s.v5[o5 - 5]);
      f5[3] = face(bc, s.v5[o5 + 5]);
      f5[4] = face(bc, s.v5[o5 - 1]);
      f5[5] = face(bc, s.v5[o5 + 1]);
      di5 = drcp(T(16) * diag5());
    }
    wave_sync();
    for (int v = lane; v < 729; v += 64) s.v9[v] = T(0);
    for (int v = lane; v < 125; v += 64) s.v5[v] = T(0);
    wave_sync();
  }
  __device__ T diag(int k) const { return ((fx[k] + fx[k + 1]) + (fym[k] + fyp[k])) + (fzm[k] + fzp[k]); }
  __device__ T diag5() const { return ((f5[0] + f5[1]) + (f5[2] + f5[3])) + (f5[4] + f5[5]); }
  // publish the column's (vertex's) values; sums of faces times neighbours
  __device__ void put9(const T (&v)[7]) {
    wave_sync();
    if (on9) {
#pragma unroll
      for (int k = 0; k < 7; ++k) s.v9[o9 + k * 81] = v[k];
    }
    wave_sync();
  }
  __device__ void put5(T v) {
    wave_sync();
    if (on5) s.v5[o5] = v;
    wave_sync();
  }
  __device__ T off(int k) const {
    const int o = o9 + k * 81;
    const T xm = k > 0 ? x[k > 0 ? k - 1 : 0] : T(0), xp = k < 6 ? x[k < 6 ? k + 1 : 0] : T(0);
    return ((fx[k] * xm + fx[k + 1] * xp) + (fym[k] * s.v9[o - 9] + fyp[k] * s.v9[o + 9])) +
           (fzm[k] * s.v9[o - 1] + fzp[k] * s.v9[o + 1]);
  }
  __device__ T off5() const {
    return ((f5[0] * s.v5[o5 - 25] + f5[1] * s.v5[o5 + 25]) +
            (f5[2] * s.v5[o5 - 5] + f5[3] * s.v5[o5 + 5])) +
           (f5[4] * s.v5[o5 - 1] + f5[5] * s.v5[o5 + 1]);
  }
  // x <- x + omega D^-1 (b - A x)
  __device__ void jac9(T om) {
    put9(x);
    T y[7];
#pragma unroll
    for (int k = 0; k < 7; ++k) y[k] = x[k] + om * ((b[k] + T(64) * off(k)) * di[k] - x[k]);
#pragma unroll
    for (int k = 0; k < 7; ++k) x[k] = y[k];
  }
  __device__ void jac5(T om) {
    put5(x5);
    x5 = x5 + om * ((b5 + T(16) * off5()) * di5 - x5);
  }
  // right-hand side of 5^3: full weighting of the 9^3 field w (zero boundary)
  __device__ void restrict9(const T (&w)[7]) {
    put9(w);
    const int i = on5 ? lane : 0;
    const int c = ((2 * (1 + i / 9)) * 9 + 2 * (1 + (i / 3) % 3)) * 9 + 2 * (1 + i % 3);
    T acc = T(0);
#pragma unroll
    for (int dx = -1; dx <= 1; ++dx) {
      T ay = T(0);
#pragma unroll
      for (int dy = -1; dy <= 1; ++dy) {
        const T* p = &s.v9[c + dx * 81 + dy * 9];
        ay += (dy == 0 ? T(0.5) : T(0.25)) * (T(0.25) * p[-1] + T(0.5) * p[0] + T(0.25) * p[1]);
      }
      acc += (dx == 0 ? T(0.5) : T(0.25)) * ay;
    }
    b5 = acc;
  }
  // the exact 3^3 solution for the full weighting of the 5^3 field w (every lane)
  __device__ T solve3(T w) {
    put5(w);
    T acc = T(0);
#pragma unroll
    for (int dx = -1; dx <= 1; ++dx) {
      T ay = T(0);
#pragma unroll
      for (int dy = -1; dy <= 1; ++dy) {
        const T* p = &s.v5[62 + dx * 25 + dy * 5];
        ay += (dy == 0 ? T(0.5) : T(0.25)) * (T(0.25) * p[-1] + T(0.5) * p[0] + T(0.25) * p[1]);
      }
      acc += (dx == 0 ? T(0.5) : T(0.25)) * ay;
    }
    return acc * di3;
  }
  // trilinear prolongation of the 3^3 value to the lane's 5^3 vertex
  __device__ T prolong3(T x3) const {
    const int i = on5 ? lane : 0;
    const T wx = i / 9 == 1 ? T(1) : T(0.5), wy = (i / 3) % 3 == 1 ? T(1) : T(0.5),
            wz = i % 3 == 1 ? T(1) : T(0.5);
    return (wx * wy * wz) * x3;
  }
  // prolongation of the 5^3 iterate to the column: added to x, or (set) as x
  __device__ void prolong5(bool set) {
    put5(x5);
    const int iy = 1 + (on9 ? lane >> 3 : 0), iz = 1 + (on9 ? lane & 7 : 0);
    const int dy = (iy & 1) ? 5 : 0, dz = iz & 1;
    const T* p = &s.v5[(iy >> 1) * 5 + (iz >> 1)];
    T w[5];
#pragma unroll
    for (int j = 0; j < 5; ++j)
      w[j] = T(0.25) * ((p[j * 25] + p[j * 25 + dz]) + (p[j * 25 + dy] + p[j * 25 + dy + dz]));
#pragma unroll
    for (int k = 0; k < 7; ++k) {
      const T v = (k & 1) ? w[(k + 1) / 2] : T(0.5) * (w[k / 2] + w[k / 2 + 1]);
      x[k] = set ? v : x[k] + v;
    }
  }
  __device__ void resid9(T (&r)[7]) {
    put9(x);
#pragma unroll
    for (int k = 0; k < 7; ++k) r[k] = b[k] - T(64) * (diag(k) * x[k] - off(k));
  }
  // the rest of a 5^3 cycle after its pre-smoothing
  __device__ void coarse5(const VsArgs& va) {
    put5(x5);
    const T r5 = b5 - T(16) * (diag5() * x5 - off5());
    x5 += prolong3(solve3(r5));
    for (int j = va.deg - 1; j >= 0; --j) jac5((T)va.om[j]);
  }
  // coarse-grid correction and post-smoothing of a 9^3 cycle after its
  // pre-smoothing: residual, a 5^3 cycle from zero, prolongation
  __device__ void coarse9(const VsArgs& va) {
    T r[7];
    resid9(r);
    restrict9(r);
    x5 = (T)va.om[0] * (b5 * di5);
    for (int j = 1; j < va.deg; ++j) jac5((T)va.om[j]);
    coarse5(va);
    prolong5(false);
    for (int j = va.deg - 1; j >= 0; --j) jac9((T)va.om[j]);
  }
  // START: the full-multigrid start of the three grids instead of a cycle from zero
  template <bool START>
  __device__ void solve(const VsArgs& va) {
    if constexpr (START) {
      // b on 5^3 and 3^3, the exact 3^3 solution, then one cycle a grid from the
      // prolonged solution of the grid below
      restrict9(b);
      x5 = prolong3(solve3(b5));
      for (int j = 0; j < va.deg; ++j) jac5((T)va.om[j]);
      coarse5(va);
      prolong5(true);
      for (int j = 0; j < va.deg; ++j) jac9((T)va.om[j]);
    } else {
#pragma unroll
      for (int k = 0; k < 7; ++k) x[k] = (T)va.om[0] * (b[k] * di[k]);
      for (int j = 1; j < va.deg; ++j) jac9((T)va.om[j]);
    }
    coarse9(va);
  }
};

// One problem of k_vsmall, by one wave.
template <typename T, int CK, bool START>
__device__ __forceinline__ void vs_problem(VsLds<T>& lds, int lane, int prob, const VsArgs& va,
                                           const T* __restrict__ b9, const void* __restrict__ c9,
                                           const void* __restrict__ c5,
                                           const void* __restrict__ c3, T* __restrict__ xout,
                                           const int* __restrict__ poff,
                                           double* __restrict__ partial) {
  using CR = typename VsWave<T, CK>::CR;
  VsWave<T, CK> w(lds, lane);
  const T* brow = b9 + (size_t)prob * 729;
#pragma unroll
  for (int k = 0; k < 7; ++k) {
    const T v = brow[w.o9 + k * 81];
    w.b[k] = w.on9 ? v : T(0);
  }
  w.load((const CR*)c9 + (size_t)prob * 729, (const CR*)c5 + (size_t)prob * 125,
         (const CR*)c3 + (size_t)prob * 27);
  w.coefficients();
  w.template solve<START>(va);
  T* xrow = xout + (size_t)prob * 729;
  if (w.on9) {
#pragma unroll
    for (int k = 0; k < 7; ++k) xrow[w.o9 + k * 81] = w.x[k];
  }
  if (partial != nullptr && prob >= va.top_begin) {
    double dot = 0.0;
    if (w.on9) {
#pragma unroll
      for (int k = 0; k < 7; ++k) dot += (double)w.b[k] * (double)w.x[k];
    }
    dot = wave_sum63(dot);
    if (lane == 63) partial[poff[prob]] = dot;
  }
}

template <typename T, int CK, bool START>
__global__ void __launch_bounds__(64 * VS_WAVES)
    k_vsmall(VsArgs va, int rows, const CgScal* __restrict__ scal, const T* __restrict__ b9,
             const void* __restrict__ c9, const void* __restrict__ c5,
             const void* __restrict__ c3, T* __restrict__ xout, const int* __restrict__ poff,
             double* __restrict__ partial) {
  __shared__ VsLds<T> lds[VS_WAVES];
  const int wave = threadIdx.x >> 6, lane = threadIdx.x & 63;
  const int prob = blockIdx.x * VS_WAVES + wave;
  if (prob >= rows || (scal && !scal[prob].active)) return;  // uniform per wave, no barriers
  vs_problem<T, CK, START>(lds[wave], lane, prob, va, b9, c9, c5, c3, xout, poff, partial);
}

// The same cycle (START: start) from 17^3 down for batches that leave the chip
// idle: one workgroup per problem, eight waves on the 17^3 grid and a ninth on
// the grids below it, in place of a pre-smoothing, a k_vsmall and a
// post-smoothing launch that each wait for their loads and form their faces
// anew.  A thread holds eight x points of a 17^3 column in registers (faces,
// right-hand side, iterate, reciprocal diagonal); LDS passes values to the
// neighbouring columns through two buffers in turn, one barrier a step.  The
// ninth wave prepares its coefficients meanwhile and runs its part between two
// barriers; both roles meet every barrier (the counts are noted at each).
// Problems whose top grid is 9^3 (rows17 and on) take a wave each, in workgroups
// that come first: they are the shorter ones, and the CUs they free take the
// 17^3 problems that did not fit at once (an objective with 231 and 932 problems
// on 17^3 and 9^3 2.89 -> 2.83 ms against the other order).
// Faces and reciprocal diagonals take the two-step reciprocal: the first step of
// a pre-smoothing pass (k_dinv) and the residual after the start's have it too.  The
// one-step form would leave up to 2.1e-15 in them (at most 1.1e-16 with two); it
// measured 1.324 against 1.348 ms on one 33^3 state and adjoint solve.
// Two register sets (the 17^3 waves' 130 and the ninth's 200) share 168 VGPRs a
// lane; the compiler keeps some thirty of the ninth wave's values in scratch.
// Gradients on one level of 17^3, 64 / 256 / 512 samples: FP64 1.31 -> 1.07,
// 1.83 -> 1.44, 2.49 -> 2.25 ms; FP32 cycles 1.28 -> 0.95, 1.68 -> 1.30,
// 2.27 -> 1.98; one 33^3 solve and adjoint 1.67 -> 1.46 ms.
constexpr int VM_FINE = 512;   // threads on the 17^3 grid
constexpr int VM_WAVES = VM_FINE / 64 + 1;
constexpr int VM_XS = 8, VM_P = 17, VM_PP = VM_P * VM_P, VM_N = VM_P * VM_PP;

template <typename T, int CK, bool START>
__global__ void __launch_bounds__(64 * VM_WAVES)
    k_vmid(VsArgs va, MidArgs<T> ma, const CgScal* __restrict__ scal,
           const int* __restrict__ poff, double* __restrict__ partial) {
  using CR = typename VsWave<T, CK>::CR;
  __shared__ T v17[2][VM_N];
  __shared__ T rb[343];             // right-hand side of 9^3
  __shared__ VsLds<T> lds;
  __shared__ double sred[VM_FINE / 64];
  const int np9 = (ma.rows9 - ma.rows17 + VM_WAVES - 1) / VM_WAVES;
  const int prob = (int)blockIdx.x < np9 ? ma.rows17 + (int)blockIdx.x : (int)blockIdx.x - np9;
  const int wave = __builtin_amdgcn_readfirstlane(threadIdx.x >> 6);
  if (prob >= ma.rows17) {
    const int pw = ma.rows17 + (prob - ma.rows17) * VM_WAVES + wave;
    if (pw >= ma.rows9 || (scal && !scal[pw].active)) return;   // uniform per wave, no barriers
    static_assert(VM_WAVES * sizeof(VsLds<T>) <= sizeof(v17), "");
    vs_problem<T, CK, START>(reinterpret_cast<VsLds<T>*>(&v17[0][0])[wave], threadIdx.x & 63, pw,
                             va, ma.b9, ma.c9, ma.c5, ma.c3, ma.x9, poff, partial);
    return;
  }
  if (scal && !scal[prob].active) return;   // uniform per workgroup
  const int npre = START ? va.deg : va.deg - 1;   // pre-smoothing steps that read neighbours

  if (wave == VM_FINE / 64) {
    const int lane = threadIdx.x & 63;
    VsWave<T, CK> w(lds, lane);
    const int rl = w.on9 ? (lane >> 3) * 7 + (lane & 7) : 0;
    auto rhs = [&] {
#pragma unroll
      for (int k = 0; k < 7; ++k) w.b[k] = w.on9 ? rb[k * 49 + rl] : T(0);
    };
    w.load((const CR*)ma.c9 + (size_t)prob * 729, (const CR*)ma.c5 + (size_t)prob * 125,
           (const CR*)ma.c3 + (size_t)prob * 27);
    __syncthreads();   // 1/a of 17^3 in LDS
    w.coefficients();
    __syncthreads();   // 17^3 faces formed
    if constexpr (START) {
      __syncthreads();   // b published
      __syncthreads();   // b of 9^3 in rb
      rhs();
      w.template solve<true>(va);
      w.put9(w.x);
      __syncthreads();   // start of 9^3 in lds.v9
    }
    for (int j = 0; j < npre + 2; ++j) __syncthreads();   // steps, x and r published
    __syncthreads();   // right-hand side of 9^3 in rb
    rhs();
    w.template solve<false>(va);
    w.put9(w.x);
    __syncthreads();   // correction of 9^3 in lds.v9
    for (int j = 0; j < va.deg; ++j) __syncthreads();   // post-smoothing
    __syncthreads();   // wave sums
    return;
  }

  const int tid = threadIdx.x;
  const int iz = tid & 15, iy = (tid >> 4) & 15, x0 = 1 + VM_XS * (tid >> 8);
  const int l0 = (x0 * VM_P + iy) * VM_P + iz;   // vertex of the first own point
  const T ih2 = T(256);
  const CR* __restrict__ c = (const CR*)ma.c17 + (size_t)prob * VM_N;
  const T* __restrict__ brow = ma.b17 + (size_t)prob * VM_N;
  T b[VM_XS], x[VM_XS], di[VM_XS];
  T fx[VM_XS + 1], fym[VM_XS], fyp[VM_XS], fzm[VM_XS], fzp[VM_XS];
  bool own[VM_XS];
#pragma unroll
  for (int j = 0; j < VM_XS; ++j) {
    own[j] = iy >= 1 && iz >= 1 && x0 + j <= 15;
    b[j] = own[j] ? brow[l0 + j * VM_PP] : T(0);
  }
  for (int v = tid; v < VM_N; v += VM_FINE) {
    v17[1][v] = VsWave<T, CK>::cvt(c[v]);
    v17[0][v] = T(0);
  }
  __syncthreads();   // 1/a in LDS
  {
    // (planes beyond the grid stand for points that are not owned)
    auto bp = [&](int j) { return &v17[1][l0 + (x0 + j <= 16 ? j : 16 - x0) * VM_PP]; };
#pragma unroll
    for (int j = 0; j <= VM_XS; ++j) fx[j] = face(*bp(j - 1), *bp(j));
#pragma unroll
    for (int j = 0; j < VM_XS; ++j) {
      const T* p = bp(j);
      fym[j] = face(p[0], p[-VM_P]);
      // (the last plane's row past the grid is the boundary row itself)
      fyp[j] = face(p[0], p[VM_P]);
      fzp[j] = face(p[0], p[1]);
      fzm[j] = __shfl_up(fzp[j], 1, 16);   // of lane iz - 1
      di[j] = drcp(ih2 * (((fx[j] + fx[j + 1]) + (fym[j] + fyp[j])) + (fzm[j] + fzp[j])));
    }
  }
  __syncthreads();   // faces formed
  for (int v = tid; v < VM_N; v += VM_FINE) v17[1][v] = T(0);
  int q = 0;
  const T* vq = nullptr;   // the values published last
  auto publish = [&](const T (&v)[VM_XS]) {   // one barrier
#pragma unroll
    for (int j = 0; j < VM_XS; ++j)
      if (own[j]) v17[q][l0 + j * VM_PP] = v[j];
    vq = &v17[q][l0];
    __syncthreads();
    q ^= 1;
  };
  // sum of faces times neighbours, x published
  const int up = x0 + VM_XS <= 16 ? VM_XS * VM_PP : 0;
  auto off = [&](int j, T lo, T hi) {
    const T xm = j > 0 ? x[j > 0 ? j - 1 : 0] : lo;
    const T xp = j < VM_XS - 1 ? x[j < VM_XS - 1 ? j + 1 : 0] : hi;
    const T* p = vq + j * VM_PP;
    return ((fx[j] * xm + fx[j + 1] * xp) + (fym[j] * p[-VM_P] + fyp[j] * p[VM_P])) +
           (fzm[j] * p[-1] + fzp[j] * p[1]);
  };
  auto jac = [&](T om) {   // x <- x + omega D^-1 (b - A x)
    publish(x);
    const T lo = vq[-VM_PP], hi = vq[up];
    T y[VM_XS];
#pragma unroll
    for (int j = 0; j < VM_XS; ++j)
      y[j] = own[j] ? x[j] + om * ((b[j] + ih2 * off(j, lo, hi)) * di[j] - x[j]) : T(0);
#pragma unroll
    for (int j = 0; j < VM_XS; ++j) x[j] = y[j];
  };
  auto restrict17 = [&](const T (&v)[VM_XS]) {   // full weighting into rb; two barriers
    publish(v);
    const T* u = vq - l0;
    if (tid < 343) {
      const int e = (2 * (1 + tid / 49) * VM_P + 2 * (1 + (tid / 7) % 7)) * VM_P + 2 * (1 + tid % 7);
      T acc = T(0);
#pragma unroll
      for (int dx = -1; dx <= 1; ++dx) {
        T ay = T(0);
#pragma unroll
        for (int dy = -1; dy <= 1; ++dy) {
          const T* p = u + e + dx * VM_PP + dy * VM_P;
          ay += (dy == 0 ? T(0.5) : T(0.25)) * (T(0.25) * p[-1] + T(0.5) * p[0] + T(0.25) * p[1]);
        }
        acc += (dx == 0 ? T(0.5) : T(0.25)) * ay;
      }
      rb[tid] = acc;
    }
    __syncthreads();
  };
  auto prolong9 = [&](bool set) {   // the 9^3 values added to x, or (set) as x
    const int dy = (iy & 1) ? 9 : 0, dz = iz & 1;
    const T* p = &lds.v9[(x0 >> 1) * 81 + (iy >> 1) * 9 + (iz >> 1)];
    T w[5];
#pragma unroll
    for (int j = 0; j < 5; ++j)
      w[j] = T(0.25) * ((p[j * 81] + p[j * 81 + dz]) + (p[j * 81 + dy] + p[j * 81 + dy + dz]));
#pragma unroll
    for (int j = 0; j < VM_XS; ++j) {
      const T v = (j & 1) ? w[(j + 1) / 2] : T(0.5) * (w[j / 2] + w[j / 2 + 1]);
      x[j] = own[j] ? (set ? v : x[j] + v) : T(0);
    }
  };
  if constexpr (START) {
    restrict17(b);      // b published, b of 9^3 in rb
    __syncthreads();    // start of 9^3 in lds.v9
    prolong9(true);
    for (int j = 0; j < va.deg; ++j) jac((T)va.om[j]);
  } else {
#pragma unroll
    for (int j = 0; j < VM_XS; ++j) x[j] = own[j] ? (T)va.om[0] * (b[j] * di[j]) : T(0);
    for (int j = 1; j < va.deg; ++j) jac((T)va.om[j]);
  }
  {
    publish(x);
    const T lo = vq[-VM_PP], hi = vq[up];
    T r[VM_XS];
#pragma unroll
    for (int j = 0; j < VM_XS; ++j) {
      const T diag = ((fx[j] + fx[j + 1]) + (fym[j] + fyp[j])) + (fzm[j] + fzp[j]);
      r[j] = own[j] ? b[j] - ih2 * (diag * x[j] - off(j, lo, hi)) : T(0);
    }
    restrict17(r);      // r published, right-hand side of 9^3 in rb
  }
  __syncthreads();      // correction of 9^3 in lds.v9
  prolong9(false);
  for (int j = va.deg - 1; j >= 0; --j) jac((T)va.om[j]);
  T* xrow = ma.x17 + (size_t)prob * VM_N;
#pragma unroll
  for (int j = 0; j < VM_XS; ++j)
    if (own[j]) xrow[l0 + j * VM_PP] = x[j];
  const bool sum = partial != nullptr && prob >= ma.top17;
  if (sum) {
    double dot = 0.0;
#pragma unroll
    for (int j = 0; j < VM_XS; ++j) dot += (double)b[j] * (double)x[j];
    dot = wave_sum63(dot);
    if ((tid & 63) == 63) sred[wave] = dot;
  }
  __syncthreads();      // wave sums
  if (sum && tid < ma.slots) {
    double t = 0.0;
#pragma unroll
    for (int w = 0; w < VM_FINE / 64; ++w) t += sred[w];
    partial[poff[prob] + tid] = tid == 0 ? t : 0.0;
  }
}

// A workgroup of k_vmid fills a CU, so its time grows by a round for every 256 of
// them (a 17^3 problem each, nine 9^3 problems each), where the separate passes
// fill the chip better and better; k_vsmall holds some twenty 9^3 problems a CU.
// FP64, gradients on 17^3 alone, separate against one kernel: 1024 samples 3.93 /
// 3.75 ms, 1536 5.61 / 5.90.  With problems topped on 9^3 (levels 9^3 and 17^3,
// M9 / M17) a first round always pays and a second only if 17^3 fills half of the
// first: 2000 / 2 1.89 / 1.73, 2300 / 2 (258 workgroups) 2.18 / 2.21, 3000 / 32
// 2.38 / 2.50, 3000 / 128 (476) 2.78 / 2.73, 3600 / 128 (543) 2.92 / 3.14, 1024 / 512
// (683) 3.18 / 3.23, 16384 / 64 7.98 / 9.82.  FP32 cycles gain up to five rounds:
// 8000 / 2 (891) 3.49 / 3.45, 4096 / 512 (1024) 3.85 / 3.69, 8000 / 256 (1173) 4.51 /
// 4.42, 10000 / 128 (1254) 4.76 / 4.68, 10000 / 256 (1396) 5.20 / 5.23, 10000 / 512
// (1681) 5.90 / 6.33, 17^3 alone 1024 3.39 / 3.20, 1536 5.15 / 5.23.
bool mid_rows(int rows17, int tops9, int elem) {
  const int packs = cdiv(tops9, VM_WAVES);
  if (rows17 > 1024) return false;
  if (packs == 0) return true;
  if (elem == 4) return rows17 + packs <= 1280;
  return rows17 + packs <= 256 || (rows17 >= 128 && rows17 + packs <= 512);
}

template <typename T>
void vcycle_mid(const double* om, int deg, int top9, const CgScal* scal, const MidArgs<T>& ma,
                int cache_bf16, const int* poff, double* partial, bool start, hipStream_t s) {
  if (ma.rows9 <= 0) return;
  VsArgs va{};
  for (int j = 0; j < deg && j < VS_MAXDEG; ++j) va.om[j] = om[j];
  va.deg = deg;
  va.top_begin = top9;
#define MLSGD_LAUNCH(CK_, START_)                                                              \
  hipLaunchKernelGGL((k_vmid<T, CK_, START_>),                                                 \
                     dim3(ma.rows17 + cdiv(ma.rows9 - ma.rows17, VM_WAVES)), dim3(64 * VM_WAVES), 0, \
                     s, va, ma, scal, poff, partial)
  if (sizeof(T) == 4 && cache_bf16) {
    if constexpr (sizeof(T) == 4) {
      if (start)
        MLSGD_LAUNCH(2, true);
      else
        MLSGD_LAUNCH(2, false);
    }
  } else if (start) {
    MLSGD_LAUNCH(1, true);
  } else {
    MLSGD_LAUNCH(1, false);
  }
#undef MLSGD_LAUNCH
}
template void vcycle_mid<double>(const double*, int, int, const CgScal*, const MidArgs<double>&, int,
                                 const int*, double*, bool, hipStream_t);
template void vcycle_mid<float>(const double*, int, int, const CgScal*, const MidArgs<float>&, int,
                                const int*, double*, bool, hipStream_t);

template <typename T>
void vcycle_small(int rows, const double* om, int deg, int top_begin, const CgScal* scal,
                  const T* b9, const void* c9, const void* c5, const void* c3, int cache_bf16,
                  T* xout, const int* poff, double* partial, bool start, hipStream_t s) {
  if (rows <= 0) return;
  VsArgs va{};
  for (int j = 0; j < deg && j < VS_MAXDEG; ++j) va.om[j] = om[j];
  va.deg = deg;
  va.top_begin = top_begin;
#define MLSGD_LAUNCH(CK_, START_)                                                             \
  hipLaunchKernelGGL((k_vsmall<T, CK_, START_>), dim3(cdiv(rows, VS_WAVES)), dim3(64 * VS_WAVES), \
                     0, s, va, rows, scal, b9, c9, c5, c3, xout, poff, partial)
  if (sizeof(T) == 4 && cache_bf16) {
    if constexpr (sizeof(T) == 4) {
      if (start)
        MLSGD_LAUNCH(2, true);
      else
        MLSGD_LAUNCH(2, false);
    }
  } else if (start) {
    MLSGD_LAUNCH(1, true);
  } else {
    MLSGD_LAUNCH(1, false);
  }
#undef MLSGD_LAUNCH
}
template void vcycle_small<double>(int, const double*, int, int, const CgScal*, const double*,
                                   const void*, const void*, const void*, int, double*, const int*,
                                   double*, bool, hipStream_t);
template void vcycle_small<float>(int, const double*, int, int, const CgScal*, const float*,
                                  const void*, const void*, const void*, int, float*, const int*,
                                  double*, bool, hipStream_t);

// ---------------------------------------------------------------------------
// Unpreconditioned CG on small grids (at most 17^3), a whole solve per
// workgroup: every vector of a 17^3 problem (27 KB) fits one CU, so one kernel
// runs all iterations where the level-by-level path makes six launches an
// iteration, each over 64 rows of 3375 unknowns and bound by its launch and by
// one march's latency.  A thread owns XS consecutive x points of one (y, z)
// column; x, r, its part of p and the faces stay in registers, the direction
// p alone in LDS for the neighbours, and the two dots of an iteration take one
// barrier each.  CgScal ends as the level-by-level path leaves it: the same
// recurrence, exit tests, iteration limit and restarts from the true residual
// (the dots' summation order differs).  64 solves of 17^3 to 1e-12 (about 100
// iterations): 3.3 ms level by level, 0.19 ms here.
// ---------------------------------------------------------------------------
// CY x CY columns (n - 2 <= CY), NS segments of XS x planes (n - 2 <= NS XS)
template <int CY, int NS, int XS>
__global__ void __launch_bounds__(CY* CY* NS)
    k_cg_small(int n, int row0, CgScal* __restrict__ scal, const double* __restrict__ cache,
               const double* __restrict__ rhs, double* __restrict__ xout, double rtol,
               int max_iters) {
  constexpr int NT = CY * CY * NS, NW = NT / 64;
  constexpr int PZ = CY + 2, PP = PZ * PZ;
  __shared__ double sp[(NS * XS + 2) * PP];   // p with its zero boundary
  __shared__ double sred[2][NW];
  const int tid = threadIdx.x;
  const int lz = tid % CY, ly = (tid / CY) % CY, seg = tid / (CY * CY);
  const int iy = 1 + ly, iz = 1 + lz, x0 = 1 + seg * XS;
  const bool col = iy <= n - 2 && iz <= n - 2;
  const int LP = lay_pitch(n), LO = lay_off(n);
  const size_t per = (size_t)lay_row(n);
  const double* __restrict__ c = cache + (size_t)(row0 + blockIdx.x) * per;
  const double* __restrict__ b = rhs + (size_t)blockIdx.x * per;
  double* __restrict__ xo = xout + (size_t)blockIdx.x * per;
  const double ih2 = (double)(n - 1) * (double)(n - 1);
  for (int i = tid; i < (NS * XS + 2) * PP; i += NT) sp[i] = 0.0;

  // faces and right-hand side of the own points (zero off the interior)
  double fx[XS + 1], fym[XS], fyp[XS], fzm[XS], fzp[XS], r[XS], x[XS], p[XS];
  auto at = [&](int ix, int jy, int jz) { return ((size_t)ix * n + jy) * LP + jz + LO; };
#pragma unroll
  for (int j = 0; j <= XS; ++j) {
    fx[j] = 0.0;
    if (col && x0 + j <= n - 1) fx[j] = face(c[at(x0 + j - 1, iy, iz)], c[at(x0 + j, iy, iz)]);
  }
  bool own[XS];
#pragma unroll
  for (int j = 0; j < XS; ++j) {
    own[j] = col && x0 + j <= n - 2;
    fym[j] = fyp[j] = fzm[j] = fzp[j] = r[j] = 0.0;
    x[j] = 0.0;
    if (own[j]) {
      const double bc = c[at(x0 + j, iy, iz)];
      fym[j] = face(bc, c[at(x0 + j, iy - 1, iz)]);
      fyp[j] = face(bc, c[at(x0 + j, iy + 1, iz)]);
      fzm[j] = face(bc, c[at(x0 + j, iy, iz - 1)]);
      fzp[j] = face(bc, c[at(x0 + j, iy, iz + 1)]);
      r[j] = b[at(x0 + j, iy, iz)];
    }
  }
  const int l0 = (x0 * PZ + iy) * PZ + iz;   // LDS slot of the first own point
  // A v at the own points, v in LDS and (own part) in registers
  auto apply = [&](const double (&v)[XS], double (&q)[XS]) {
    const double lo = sp[l0 - PP], hi = sp[l0 + XS * PP];
#pragma unroll
    for (int j = 0; j < XS; ++j) {
      const double xm = j > 0 ? v[j > 0 ? j - 1 : 0] : lo;
      const double xp = j < XS - 1 ? v[j < XS - 1 ? j + 1 : 0] : hi;
      const int l = l0 + j * PP;
      const double diag = ((fx[j] + fx[j + 1]) + (fym[j] + fyp[j])) + (fzm[j] + fzp[j]);
      const double off = ((fx[j] * xm + fx[j + 1] * xp) +
                          (fym[j] * sp[l - PZ] + fyp[j] * sp[l + PZ])) +
                         (fzm[j] * sp[l - 1] + fzp[j] * sp[l + 1]);
      q[j] = own[j] ? ih2 * (diag * v[j] - off) : 0.0;
    }
  };
  auto publish = [&](const double (&v)[XS]) {   // own values into LDS
#pragma unroll
    for (int j = 0; j < XS; ++j)
      if (own[j]) sp[l0 + j * PP] = v[j];
  };
  int slot = 0;
  // sum over the workgroup, known to every thread; one barrier (two slots in
  // turn: a slot is written again only after the other sum's barrier)
  auto total = [&](double v) {
    v = wave_sum63(v);
    if ((tid & 63) == 63) sred[slot][tid >> 6] = v;
    __syncthreads();
    double t = 0.0;
#pragma unroll
    for (int w = 0; w < NW; ++w) t += sred[slot][w];
    slot ^= 1;
    return t;
  };
  auto norm2 = [&](const double (&v)[XS]) {
    double t = 0.0;
#pragma unroll
    for (int j = 0; j < XS; ++j) t += v[j] * v[j];
    return total(t);
  };
  __syncthreads();   // sp is cleared

  const double rt2 = rtol * rtol;
  const double bb = norm2(r);
  double rr = bb;
  int iters = 0, again = 0;
  bool active = bb > 0.0;
  for (int restart = 0; restart < 3 && active; ++restart) {
    double rz = rr;
#pragma unroll
    for (int j = 0; j < XS; ++j) p[j] = r[j];
    publish(p);
    __syncthreads();
    while (active) {
      double q[XS];
      apply(p, q);
      double t = 0.0;
#pragma unroll
      for (int j = 0; j < XS; ++j) t += p[j] * q[j];
      const double pq = total(t);
      if (!(pq > 0.0)) break;
      const double alpha = rz / pq;
#pragma unroll
      for (int j = 0; j < XS; ++j) {
        x[j] += alpha * p[j];
        r[j] -= alpha * q[j];
      }
      rr = norm2(r);
      ++iters;
      if (!(rr > rt2 * bb) || iters >= max_iters) break;
      const double beta = rr / rz;
      rz = rr;
#pragma unroll
      for (int j = 0; j < XS; ++j) p[j] = r[j] + beta * p[j];
      publish(p);
      __syncthreads();
    }
    // the true residual b - A x decides; a problem that drifted starts again
    publish(x);
    __syncthreads();
    double q[XS];
    apply(x, q);
#pragma unroll
    for (int j = 0; j < XS; ++j)
      r[j] = own[j] ? b[at(x0 + j, iy, iz)] - q[j] : 0.0;
    rr = norm2(r);
    active = rr > rt2 * bb && iters < max_iters;
    again = active;
  }
#pragma unroll
  for (int j = 0; j < XS; ++j)
    if (own[j]) xo[at(x0 + j, iy, iz)] = x[j];
  if (tid == 0) {
    CgScal sc{};
    sc.bb = bb;
    sc.rr = rr;
    sc.iters = iters;
    sc.active = sc.restart = again;
    scal[row0 + blockIdx.x] = sc;
  }
}

void cg_small(int n, int rows, int row0, CgScal* scal, const double* cache, const double* rhs,
              double* x, double rtol, int max_iters, hipStream_t s) {
  if (rows <= 0) return;
#define MLSGD_LAUNCH(CY_, NS_, XS_)                                                             \
  hipLaunchKernelGGL((k_cg_small<CY_, NS_, XS_>), dim3(rows), dim3(CY_ * CY_ * NS_), 0, s, n, row0, \
                     scal, cache, rhs, x, rtol, max_iters)
  if (n <= 6)
    MLSGD_LAUNCH(4, 4, 1);
  else if (n <= 10)
    MLSGD_LAUNCH(8, 2, 4);
  else
    MLSGD_LAUNCH(16, 4, 4);
#undef MLSGD_LAUNCH
}

// Reciprocal diagonal drcp(h^-2 ((fxm + fxp) + (fym + fyp)) + (fzm + fzp)) of
// every interior vertex of every row of every grid size, with the faces and the
// summation order of k_march.  One launch for all sizes, as for the coefficient
// caches it reads (k_coef_cache); a workgroup takes DINV_CHUNK elements of a row,
// with 32-bit coordinates.
constexpr int DINV_CHUNK = 256 * 8;

template <typename T, int CK>
__global__ void __launch_bounds__(256) k_dinv(FieldTable ft) {
  int k = 0;
  while (k + 1 < ft.count && blockIdx.x >= (unsigned)ft.lv[k + 1].dblk0) ++k;   // uniform
  const FieldLvl& L = ft.lv[k];
  const int n = L.n, LP = lay_pitch(n), LO = lay_off(n);
  const uint32_t per = (uint32_t)lay_row(n);
  const int blk = (int)blockIdx.x - L.dblk0;
  const int row = blk / L.dper;
  const uint32_t e0 = (uint32_t)(blk - row * L.dper) * DINV_CHUNK;
  const T* c = (const T*)(sizeof(T) == 8 ? (const void*)L.c64 : (const void*)L.c32) + (size_t)row * per;
  const uint16_t* c16 = L.c16 + (size_t)row * per;
  T* __restrict__ dinv = (T*)L.dinv + (size_t)row * per;
  const T ih2 = (T)((double)(n - 1) * (double)(n - 1));
  auto bval = [&](uint32_t e) -> T {
    if constexpr (CK == 2)
      return (T)from_bf16(c16[e]);
    else
      return c[e];
  };
  const uint32_t sx = (uint32_t)n * LP, sy = LP;
#pragma unroll 2
  for (uint32_t e = e0 + threadIdx.x; e < min(e0 + DINV_CHUNK, per); e += 256) {
    const uint32_t ix = e / sx, r = e - ix * sx, iy = r / sy;
    const int iz = (int)(r - iy * sy) - LO;
    T d = T(0);
    if (ix >= 1 && iy >= 1 && iz >= 1 && (int)ix <= n - 2 && (int)iy <= n - 2 && iz <= n - 2) {
      const T bc = bval(e);
      const T fxm = face(bval(e - sx), bc), fxp = face(bc, bval(e + sx));
      const T fym = face(bc, bval(e - sy)), fyp = face(bc, bval(e + sy));
      const T fzm = face(bc, bval(e - 1)), fzp = face(bc, bval(e + 1));
      d = drcp(ih2 * (((fxm + fxp) + (fym + fyp)) + (fzm + fzp)));
    }
    dinv[e] = d;
  }
}

// ---------------------------------------------------------------------------
// Fused red-black Gauss-Seidel sweep (both colours in one pass, out of place).
//
// x_out = GS_second(GS_first(x_in)) with relaxation omega, where x_in is the
// previous iterate (zero on a zero start) plus, optionally, the trilinear
// prolongation of a coarse correction folded into every load.  The pass is a
// wavefront along x: at plane s the first colour is updated on the patch and
// on a one-point ring around it (the ring values belong to neighbouring
// patches and are recomputed here from the same inputs, so every patch sees
// identical values), then the second colour is updated on plane s-1 of the
// patch and written out.  LDS holds three planes (values and 1/a) with a
// two-point ring; each thread keeps its own column's planes s-2..s+1 in
// registers, and threads below 2(TY+TZ)+4 also own one ring column and one
// outer-ring slot.  The coefficient is read from the per-estimate cache.
// ---------------------------------------------------------------------------
template <typename T, int TY, int TZ, bool XZERO, bool PROLONG>
__global__ void __launch_bounds__(TY* TZ)
    k_rbsweep(GridArgs g, const T* __restrict__ xin, const T* __restrict__ xc,
              const T* __restrict__ rhs, T* __restrict__ xout, int first_color,
              const int* __restrict__ poff, double* __restrict__ partial, int top_begin,
              T omega) {
  constexpr int NT = TY * TZ;
  constexpr int PZ = TZ + 4;
  constexpr int PLANE = (TY + 4) * PZ;
  constexpr int NRING = 2 * (TZ + 2) + 2 * TY;   // one-point ring incl. its 4 corners
  constexpr int NR2 = 2 * (TZ + TY);             // two-point ring without corners
  static_assert(NRING <= NT && NR2 <= NT, "tile too small for its rings");
  __shared__ T sv[3][PLANE];
  __shared__ T sb[3][PLANE];
  __shared__ double sred[NT / 64];

  const int n = g.n;
  const int LP = lay_pitch(n), LO = lay_off(n);
  const int nn = n * LP;
  const int nc = (n - 1) / 2 + 1;
  const int bid = xcd_swizzle(blockIdx.x, gridDim.x);
  const int tpr = g.t.tiles_per_row;
  const int row = bid / tpr;
  const int tile = bid - row * tpr;
  int tt = tile;
  const int ty = tt % g.t.nty;
  tt /= g.t.nty;
  const int tz = tt % g.t.ntz;
  const int xcix = tt / g.t.ntz;
  const int prob = g.row0 + row;
  if (g.scal && !g.scal[prob].active) return;  // uniform per workgroup

  const size_t stride = (size_t)g.stride;
  const T* __restrict__ xr = xin + (size_t)row * stride;
  const T* __restrict__ br = rhs + (size_t)row * stride;
  T* __restrict__ outr = xout + (size_t)row * stride;
  const T* __restrict__ cache = (const T*)g.cache + (size_t)prob * stride;
  const T* __restrict__ xcr = PROLONG ? xc + (size_t)row * (size_t)lay_row(nc) : nullptr;
  const int tid = threadIdx.x;
  const int y0 = 1 + ty * TY, z0 = 1 + tz * TZ;
  const int c1 = first_color ^ 1;

  // own tile position
  const int ly = tid / TZ, lz = tid - (tid / TZ) * TZ;
  const int oy = y0 + ly, oz = z0 + lz;
  const int oidx = (ly + 2) * PZ + (lz + 2);
  // one-point ring column (LDS coordinates in [1, TY+2] x [1, TZ+2])
  int rly = 0, rlz = 0;
  if (tid < NRING) {
    if (tid < TZ + 2) {
      rly = 1; rlz = tid + 1;
    } else if (tid < 2 * (TZ + 2)) {
      rly = TY + 2; rlz = tid - (TZ + 2) + 1;
    } else if (tid < 2 * (TZ + 2) + TY) {
      rly = tid - 2 * (TZ + 2) + 2; rlz = 1;
    } else {
      rly = tid - 2 * (TZ + 2) - TY + 2; rlz = TZ + 2;
    }
  }
  const int ry = y0 - 2 + rly, rz = z0 - 2 + rlz;
  const int ridx = rly * PZ + rlz;
  const bool ring_corner = (rly == 1 || rly == TY + 2) && (rlz == 1 || rlz == TZ + 2);
  // two-point ring slot
  int qly = 0, qlz = 0;
  if (tid < NR2) {
    if (tid < TZ) {
      qly = 0; qlz = tid + 2;
    } else if (tid < 2 * TZ) {
      qly = TY + 3; qlz = tid - TZ + 2;
    } else if (tid < 2 * TZ + TY) {
      qly = tid - 2 * TZ + 2; qlz = 0;
    } else {
      qly = tid - 2 * TZ - TY + 2; qlz = TZ + 3;
    }
  }
  const int qy = y0 - 2 + qly, qz = z0 - 2 + qlz;
  const int qidx = qly * PZ + qlz;

  // column properties: inside the grid (coefficient exists), interior (unknown)
  const bool own_grid = oy <= n - 1 && oz <= n - 1;
  const bool own_int = oy <= n - 2 && oz <= n - 2;
  const bool ring_on = tid < NRING && ry >= 0 && rz >= 0 && ry <= n - 1 && rz <= n - 1;
  const bool ring_upd = ring_on && !ring_corner && ry >= 1 && rz >= 1 && ry <= n - 2 && rz <= n - 2;
  const bool r2_on = tid < NR2 && qy >= 0 && qz >= 0 && qy <= n - 1 && qz <= n - 1;
  const bool r2_int = r2_on && qy >= 1 && qz >= 1 && qy <= n - 2 && qz <= n - 2;
  const int ocol = oy * LP + oz + LO, rcol = ry * LP + rz + LO, qcol = qy * LP + qz + LO;
  const int opar = (oy + oz) & 1, rpar = (ry + rz) & 1;

  // previous iterate (+ prolonged coarse correction) on plane ix of a column
  auto ldx = [&](int ix, bool colint, int col, int jy, int jz) -> T {
    if (XZERO || !colint || ix < 1 || ix > n - 2) return T(0);
    T v = xr[ix * nn + col];
    if (PROLONG) v += prolong_val<T>(nc, xcr, ix, jy, jz);
    return v;
  };
  auto ldb = [&](int ix, bool colin, int col) -> T {
    if (!colin || ix < 0 || ix > n - 1) return T(1);
    return cache[ix * nn + col];
  };
  const T ih2 = (T)g.ih2;

  const int x0 = 1 + xcix * g.t.xchunk;
  const int x1 = min(x0 + g.t.xchunk, n - 1);

  // own column queue: values at s-2 .. s+1 and 1/a at s-2 .. s+1
  const int s0 = x0 - 1;
  T q0 = T(0), q1 = ldx(s0 - 1, own_int, ocol, oy, oz), q2 = ldx(s0, own_int, ocol, oy, oz),
    q3 = ldx(s0 + 1, own_int, ocol, oy, oz);
  T b0 = T(1), b1 = ldb(s0 - 1, own_grid, ocol), b2 = ldb(s0, own_grid, ocol),
    b3 = ldb(s0 + 1, own_grid, ocol);
  // ring column queue: old values and 1/a at s-1 .. s+1
  const bool rint = ring_on && ry >= 1 && rz >= 1 && ry <= n - 2 && rz <= n - 2;
  T r0 = ldx(s0 - 1, rint, rcol, ry, rz), r1 = ldx(s0, rint, rcol, ry, rz),
    r2 = ldx(s0 + 1, rint, rcol, ry, rz);
  T rb0 = ldb(s0 - 1, ring_on, rcol), rb1 = ldb(s0, ring_on, rcol), rb2 = ldb(s0 + 1, ring_on, rcol);
  // outer-ring slot: plane s
  T qv = ldx(s0, r2_int, qcol, qy, qz), qb = ldb(s0, r2_on, qcol);
  // right-hand sides: own column at s (first colour) and s-1 (second colour), ring at s
  auto ldr = [&](int ix, bool colint, int col) -> T {
    if (!colint || ix < 1 || ix > n - 2) return T(0);
    return br[ix * nn + col];
  };
  T bo_s = ldr(s0, own_int, ocol), bo_m = ldr(s0 - 1, own_int, ocol);
  T br_s = ldr(s0, ring_upd, rcol);
  double dot = 0.0;
  const bool want_dot = partial != nullptr && prob >= top_begin;

  for (int s = s0; s <= x1; ++s) {
    const int buf = (s - s0) % 3;
    const int pbuf = (s - s0 + 2) % 3;   // plane s-1
    // prefetch: columns at s+2, outer ring at s+1, right-hand sides at s+1
    const T nq = ldx(s + 2, own_int, ocol, oy, oz);
    const T nb = ldb(s + 2, own_grid, ocol);
    const T nr = ldx(s + 2, rint, rcol, ry, rz);
    const T nrb = ldb(s + 2, ring_on, rcol);
    const T nqv = ldx(s + 1, r2_int, qcol, qy, qz);
    const T nqb = ldb(s + 1, r2_on, qcol);
    const T nbo = ldr(s + 1, own_int, ocol);
    const T nbr = ldr(s + 1, ring_upd, rcol);

    // plane s (old values) into LDS
    sv[buf][oidx] = q2;
    sb[buf][oidx] = b2;
    if (tid < NRING) {
      sv[buf][ridx] = r1;
      sb[buf][ridx] = rb1;
    }
    if (tid < NR2) {
      sv[buf][qidx] = qv;
      sb[buf][qidx] = qb;
    }
    __syncthreads();
    const int spar = s & 1;
    // first colour on plane s: patch and ring (writes only first-colour
    // points, reads only second-colour neighbours: no barrier needed)
    if (own_int && s >= 1 && s <= n - 2 && (spar ^ opar) == first_color) {
      const T bc = b2;
      const T fxm = face(bc, b1), fxp = face(bc, b3);
      const T fym = face(bc, sb[buf][oidx - PZ]), fyp = face(bc, sb[buf][oidx + PZ]);
      const T fzm = face(bc, sb[buf][oidx - 1]), fzp = face(bc, sb[buf][oidx + 1]);
      const T diag = ((fxm + fxp) + (fym + fyp)) + (fzm + fzp);
      const T off = ((fxm * q1 + fxp * q3) + (fym * sv[buf][oidx - PZ] + fyp * sv[buf][oidx + PZ])) +
                    (fzm * sv[buf][oidx - 1] + fzp * sv[buf][oidx + 1]);
      const T gs = (bo_s + ih2 * off) * drcp(ih2 * diag);
      q2 = q2 + omega * (gs - q2);
      sv[buf][oidx] = q2;
    }
    if (ring_upd && s >= 1 && s <= n - 2 && (spar ^ rpar) == first_color) {
      const T bc = rb1;
      const T fxm = face(bc, rb0), fxp = face(bc, rb2);
      const T fym = face(bc, sb[buf][ridx - PZ]), fyp = face(bc, sb[buf][ridx + PZ]);
      const T fzm = face(bc, sb[buf][ridx - 1]), fzp = face(bc, sb[buf][ridx + 1]);
      const T diag = ((fxm + fxp) + (fym + fyp)) + (fzm + fzp);
      const T off = ((fxm * r0 + fxp * r2) + (fym * sv[buf][ridx - PZ] + fyp * sv[buf][ridx + PZ])) +
                    (fzm * sv[buf][ridx - 1] + fzp * sv[buf][ridx + 1]);
      const T gs = (br_s + ih2 * off) * drcp(ih2 * diag);
      sv[buf][ridx] = r1 + omega * (gs - r1);
    }
    // second colour on plane s-1 of the patch (its first-colour neighbours
    // on plane s-1 were published by the previous plane's barrier; plane s
    // is the thread's own q2), then write plane s-1 out
    const int sm1 = s - 1;
    if (own_int && sm1 >= x0 && sm1 <= x1 - 1) {
      T val = q1;
      if ((((sm1 & 1) ^ opar)) == c1) {
        const T bc = b1;
        const T fxm = face(bc, b0), fxp = face(bc, b2);
        const T fym = face(bc, sb[pbuf][oidx - PZ]), fyp = face(bc, sb[pbuf][oidx + PZ]);
        const T fzm = face(bc, sb[pbuf][oidx - 1]), fzp = face(bc, sb[pbuf][oidx + 1]);
        const T diag = ((fxm + fxp) + (fym + fyp)) + (fzm + fzp);
        const T off = ((fxm * q0 + fxp * q2) + (fym * sv[pbuf][oidx - PZ] + fyp * sv[pbuf][oidx + PZ])) +
                      (fzm * sv[pbuf][oidx - 1] + fzp * sv[pbuf][oidx + 1]);
        const T gs = (bo_m + ih2 * off) * drcp(ih2 * diag);
        val = q1 + omega * (gs - q1);
      }
      outr[sm1 * nn + ocol] = val;
      if (want_dot) dot += (double)bo_m * (double)val;
      q1 = val;
    }
    // rotate
    q0 = q1; q1 = q2; q2 = q3; q3 = nq;
    b0 = b1; b1 = b2; b2 = b3; b3 = nb;
    r0 = r1; r1 = r2; r2 = nr;
    rb0 = rb1; rb1 = rb2; rb2 = nrb;
    qv = nqv; qb = nqb;
    bo_m = bo_s; bo_s = nbo; br_s = nbr;
  }
  if (want_dot) {
    const double sum = block_sum<NT>(dot, sred);
    if (threadIdx.x == 0) partial[poff[prob] + tile] = sum;
  }
}

template <typename T>
void rb_sweep(const GridArgs& g, const T* xin, const T* xc, const T* b, T* xout, int first_color,
              int x_zero, const int* poff, double* partial, int top_begin, double omega,
              hipStream_t s) {
  if (g.rows <= 0) return;
  const int nblk = g.rows * g.t.tiles_per_row;
#define MLSGD_LAUNCH4(TY_, TZ_, XZ_, PR_)                                                   \
  hipLaunchKernelGGL((k_rbsweep<T, TY_, TZ_, XZ_, PR_>), dim3(nblk), dim3(TY_ * TZ_), 0, s, g, \
                     xin, xc, b, xout, first_color, poff, partial, top_begin, (T)omega)
#define MLSGD_LAUNCH(TY_, TZ_)                 \
  if (x_zero)                                  \
    MLSGD_LAUNCH4(TY_, TZ_, true, false);      \
  else if (xc)                                 \
    MLSGD_LAUNCH4(TY_, TZ_, false, true);      \
  else                                         \
    MLSGD_LAUNCH4(TY_, TZ_, false, false)
  if (g.t.TZ == 8) {
    MLSGD_LAUNCH(8, 8);
  } else if (g.t.TZ == 16) {
    MLSGD_LAUNCH(16, 16);
  } else if (g.t.TZ == 32) {
    MLSGD_LAUNCH(8, 32);
  } else if (g.t.TY == 8) {
    MLSGD_LAUNCH(8, 64);
  } else {
    MLSGD_LAUNCH(4, 64);
  }
#undef MLSGD_LAUNCH
#undef MLSGD_LAUNCH4
}
template void rb_sweep<double>(const GridArgs&, const double*, const double*, const double*,
                               double*, int, int, const int*, double*, int, double, hipStream_t);
template void rb_sweep<float>(const GridArgs&, const float*, const float*, const float*, float*,
                              int, int, const int*, double*, int, double, hipStream_t);

// Per-estimate cache of the reciprocal coefficient 1/a = exp(-log a) at every
// vertex of every row of every grid size.  A thread owns one (y, z) column:
// S[k1] = sum_{k2,k3} c[k1,k2,k3] cos(pi k2 y) cos(pi k3 z) once, then K FMAs and
// one FP64 exp per vertex along its x chunk (the KL sum written separably).  The
// FP64 and/or FP32 copies are written in the same pass.  One launch covers all
// grid sizes, and the columns are cut in x where the batch leaves the chip idle:
// per grid and whole lines, the four grids of one 33^3 solve took 54 us.
__global__ void __launch_bounds__(256)
    k_coef_cache(FieldTable ft, const double* __restrict__ coef, int K) {
  __shared__ double sc[KMAX * KMAX * KMAX];
  int lk = 0;
  while (lk + 1 < ft.count && blockIdx.x >= (unsigned)ft.lv[lk + 1].cblk0) ++lk;   // uniform
  const FieldLvl& L = ft.lv[lk];
  const int n = L.n;
  const double* __restrict__ cosT = L.cosT;
  const int cols = n * n;
  const int cpb = (cols + 255) / 256;
  const int blk = (int)blockIdx.x - L.cblk0;
  const int xc = blk % L.nxc, rb = blk / L.nxc;
  const int row = rb / cpb;
  const int col = (rb - row * cpb) * 256 + threadIdx.x;
  const int K3 = K * K * K;
  for (int j = threadIdx.x; j < K3; j += 256) sc[j] = coef[(size_t)row * K3 + j];
  __syncthreads();
  if (col >= cols) return;
  const int iy = col / n, iz = col - (col / n) * n;
  double S[KMAX];
#pragma unroll
  for (int k1 = 0; k1 < KMAX; ++k1) {
    double acc = 0.0;
    if (k1 < K) {
      for (int k2 = 0; k2 < K; ++k2) {
        double t = 0.0;
        for (int k3 = 0; k3 < K; ++k3) t += sc[(k1 * K + k2) * K + k3] * cosT[k3 * n + iz];
        acc += t * cosT[k2 * n + iy];
      }
    }
    S[k1] = acc;
  }
  const int LP = lay_pitch(n);
  const size_t base = (size_t)row * (size_t)lay_row(n) + (size_t)iy * LP + iz + lay_off(n);
  const int x0 = xc * L.xch, x1 = min(n, x0 + L.xch);
  for (int ix = x0; ix < x1; ++ix) {
    double l = 0.0;
#pragma unroll
    for (int k = 0; k < KMAX; ++k)
      if (k < K) l += cosT[k * n + ix] * S[k];
    const double b = exp(-l);
    const size_t i = base + (size_t)ix * n * LP;
    if (L.c64) L.c64[i] = b;
    if (L.c32) L.c32[i] = (float)b;
    if (L.c16) L.c16[i] = to_bf16((float)b);
  }
}

// ---------------------------------------------------------------------------
// Batched grid transfers.  Full weighting R = P^T / 8 (weights 1/4, 1/2, 1/4
// per axis) from fine interior to coarse interior, and trilinear
// prolongation added onto the fine rows.  Coarse boundary entries are zero.
// ---------------------------------------------------------------------------
template <typename T>
__global__ void k_restrict_rows(int nf, int rows, int row0, const CgScal* scal,
                                const T* __restrict__ fine, T* __restrict__ coarse) {
  const int nc = (nf - 1) / 2 + 1, mc = nc - 2;
  const long long per = (long long)mc * mc * mc;
  const long long total = per * rows;
  const size_t sf = (size_t)lay_row(nf), scs = (size_t)lay_row(nc);
  const int fp = lay_pitch(nf), fo = lay_off(nf), cp = lay_pitch(nc), co = lay_off(nc);
  for (long long i = (long long)blockIdx.x * blockDim.x + threadIdx.x; i < total;
       i += (long long)gridDim.x * blockDim.x) {
    const int row = (int)(i / per);
    if (scal && !scal[row0 + row].active) continue;
    const int r = (int)(i - (long long)row * per);
    const int jx = 1 + r / (mc * mc), jy = 1 + (r / mc) % mc, jz = 1 + r % mc;
    const T* f = fine + (size_t)row * sf;
    T acc = T(0);
#pragma unroll
    for (int dx = -1; dx <= 1; ++dx) {
      const T wx = dx == 0 ? T(0.5) : T(0.25);
      T ay = T(0);
#pragma unroll
      for (int dy = -1; dy <= 1; ++dy) {
        const T wy = dy == 0 ? T(0.5) : T(0.25);
        const T* p = f + ((size_t)(2 * jx + dx) * nf + (2 * jy + dy)) * fp + 2 * jz + fo;
        ay += wy * (T(0.25) * p[-1] + T(0.5) * p[0] + T(0.25) * p[1]);
      }
      acc += wx * ay;
    }
    coarse[(size_t)row * scs + ((size_t)jx * nc + jy) * cp + jz + co] = acc;
  }
}

// The y and z parts of full weighting after the pre-smoothing pass's x part: coarse vertex
// (I, J, K) = sum over dy of w(dy) (h(I, 2J+dy, 2K-1) / 4 + h(I, 2J+dy, 2K) / 2
// + h(I, 2J+dy, 2K+1) / 4), w = 1/2 at dy = 0 and 1/4 at dy = +-1, with h
// plane I held in plane I of the fine row.
template <typename T>
__global__ void k_restrict_yz_rows(int nf, int rows, int row0, const CgScal* scal,
                                   const T* __restrict__ h, T* __restrict__ coarse) {
  const int nc = (nf - 1) / 2 + 1, mc = nc - 2;
  const long long per = (long long)mc * mc * mc;
  const long long total = per * rows;
  const size_t sf = (size_t)lay_row(nf), scs = (size_t)lay_row(nc);
  const int fp = lay_pitch(nf), fo = lay_off(nf), cp = lay_pitch(nc), co = lay_off(nc);
  for (long long i = (long long)blockIdx.x * blockDim.x + threadIdx.x; i < total;
       i += (long long)gridDim.x * blockDim.x) {
    const int row = (int)(i / per);
    if (scal && !scal[row0 + row].active) continue;
    const int r = (int)(i - (long long)row * per);
    const int jx = 1 + r / (mc * mc), jy = 1 + (r / mc) % mc, jz = 1 + r % mc;
    const T* f = h + (size_t)row * sf;
    T acc = T(0);
#pragma unroll
    for (int dy = -1; dy <= 1; ++dy) {
      const T wy = dy == 0 ? T(0.5) : T(0.25);
      const T* p = f + ((size_t)jx * nf + (2 * jy + dy)) * fp + 2 * jz + fo;
      acc += wy * (T(0.25) * p[-1] + T(0.5) * p[0] + T(0.25) * p[1]);
    }
    coarse[(size_t)row * scs + ((size_t)jx * nc + jy) * cp + jz + co] = acc;
  }
}

template <typename T>
__global__ void k_prolong_add_rows(int nc, int rows, int row0, const CgScal* scal,
                                   const T* __restrict__ coarse, T* __restrict__ fine, int set) {
  const int nf = 2 * (nc - 1) + 1, mf = nf - 2;
  const long long per = (long long)mf * mf * mf;
  const long long total = per * rows;
  const size_t sf = (size_t)lay_row(nf), scs = (size_t)lay_row(nc);
  const int fp = lay_pitch(nf), fo = lay_off(nf), cp = lay_pitch(nc), co = lay_off(nc);
  for (long long i = (long long)blockIdx.x * blockDim.x + threadIdx.x; i < total;
       i += (long long)gridDim.x * blockDim.x) {
    const int row = (int)(i / per);
    if (scal && !scal[row0 + row].active) continue;
    const int r = (int)(i - (long long)row * per);
    const int ix = 1 + r / (mf * mf), iy = 1 + (r / mf) % mf, iz = 1 + r % mf;
    const T* c = coarse + (size_t)row * scs;
    const int ax = ix >> 1, bx = (ix + 1) >> 1;
    const int ay = iy >> 1, by = (iy + 1) >> 1;
    const int az = iz >> 1, bz = (iz + 1) >> 1;
    const T wx = (ix & 1) ? T(0.5) : T(1), wy = (iy & 1) ? T(0.5) : T(1),
            wz = (iz & 1) ? T(0.5) : T(1);
    auto cv = [&](int a, int b, int d) { return c[((size_t)a * nc + b) * cp + d + co]; };
    T v = cv(ax, ay, az);
    if (iz & 1) v += cv(ax, ay, bz);
    if (iy & 1) {
      v += cv(ax, by, az);
      if (iz & 1) v += cv(ax, by, bz);
    }
    if (ix & 1) {
      v += cv(bx, ay, az);
      if (iz & 1) v += cv(bx, ay, bz);
      if (iy & 1) {
        v += cv(bx, by, az);
        if (iz & 1) v += cv(bx, by, bz);
      }
    }
    T* dst = &fine[(size_t)row * sf + ((size_t)ix * nf + iy) * fp + iz + fo];
    if (set)
      *dst = wx * wy * wz * v;
    else
      *dst += wx * wy * wz * v;
  }
}

static int grid_for(long long total, int bs) {
  long long b = (total + bs - 1) / bs;
  if (b > 65536LL * 8) b = 65536LL * 8;
  if (b < 1) b = 1;
  return (int)b;
}

void field_caches(FieldTable& ft, const double* coef, int K, hipStream_t s) {
  long long cols = 0;   // workgroups of whole columns
  for (int k = 0; k < ft.count; ++k)
    cols += (long long)ft.lv[k].rows * cdiv((long long)ft.lv[k].n * ft.lv[k].n, 256);
  long long cb = 0, db = 0;
  bool d64 = false, d32 = false, d16 = false;
  for (int k = 0; k < ft.count; ++k) {
    FieldLvl& L = ft.lv[k];
    // 2048 workgroups fill the chip; chunks of at least 4 planes
    L.xch = cols >= 1024 ? L.n : std::max(4, (int)cdiv(L.n * std::max(cols, 1LL), 2048));
    L.nxc = cdiv(L.n, L.xch);
    L.cblk0 = (int)cb;
    cb += (long long)L.rows * cdiv((long long)L.n * L.n, 256) * L.nxc;
    L.dper = L.dinv ? cdiv(lay_row(L.n), DINV_CHUNK) : 0;
    L.dblk0 = (int)db;
    db += (long long)L.rows * L.dper;
    if (L.dinv) {
      if (L.c16) d16 = true;
      else if (L.c32) d32 = true;
      else d64 = true;
    }
  }
  if (std::max(cb, db) > MAX_WG256 && ft.count > 1) {
    const int half = ft.count / 2;
    FieldTable lo{}, hi{};
    for (int k = 0; k < ft.count; ++k) {
      FieldTable& h = k < half ? lo : hi;
      h.lv[h.count++] = ft.lv[k];
    }
    field_caches(lo, coef, K, s);
    field_caches(hi, coef, K, s);
    return;
  }
  if (cb > 0)
    hipLaunchKernelGGL(k_coef_cache, dim3((unsigned)cb), dim3(256), 0, s, ft, coef, K);
  if (db <= 0) return;
  if (d16)
    hipLaunchKernelGGL((k_dinv<float, 2>), dim3((unsigned)db), dim3(256), 0, s, ft);
  else if (d32)
    hipLaunchKernelGGL((k_dinv<float, 1>), dim3((unsigned)db), dim3(256), 0, s, ft);
  else if (d64)
    hipLaunchKernelGGL((k_dinv<double, 1>), dim3((unsigned)db), dim3(256), 0, s, ft);
}

template <typename T>
void restrict_rows(int nf, int rows, int row0, const CgScal* scal, const T* fine, T* coarse,
                   hipStream_t s) {
  if (rows <= 0) return;
  const int mc = (nf - 1) / 2 - 1;
  const long long total = (long long)mc * mc * mc * rows;
  hipLaunchKernelGGL(k_restrict_rows<T>, dim3(grid_for(total, 256)), dim3(256), 0, s, nf, rows,
                     row0, scal, fine, coarse);
}
template <typename T>
void restrict_yz_rows(int nf, int rows, int row0, const CgScal* scal, const T* h, T* coarse,
                      hipStream_t s) {
  if (rows <= 0) return;
  const int mc = (nf - 1) / 2 - 1;
  const long long total = (long long)mc * mc * mc * rows;
  hipLaunchKernelGGL(k_restrict_yz_rows<T>, dim3(grid_for(total, 256)), dim3(256), 0, s, nf,
                     rows, row0, scal, h, coarse);
}
template void restrict_yz_rows<double>(int, int, int, const CgScal*, const double*, double*,
                                       hipStream_t);
template void restrict_yz_rows<float>(int, int, int, const CgScal*, const float*, float*,
                                      hipStream_t);
template <typename T>
void prolong_add_rows(int nc, int rows, int row0, const CgScal* scal, const T* coarse, T* fine,
                      hipStream_t s) {
  if (rows <= 0) return;
  const int mf = 2 * (nc - 1) - 1;
  const long long total = (long long)mf * mf * mf * rows;
  hipLaunchKernelGGL(k_prolong_add_rows<T>, dim3(grid_for(total, 256)), dim3(256), 0, s, nc,
                     rows, row0, scal, coarse, fine, 0);
}
template <typename T>
void prolong_rows(int nc, int rows, const T* coarse, T* fine, hipStream_t s) {
  if (rows <= 0) return;
  const int mf = 2 * (nc - 1) - 1;
  const long long total = (long long)mf * mf * mf * rows;
  hipLaunchKernelGGL(k_prolong_add_rows<T>, dim3(grid_for(total, 256)), dim3(256), 0, s, nc,
                     rows, 0, nullptr, coarse, fine, 1);
}
template void prolong_rows<double>(int, int, const double*, double*, hipStream_t);
template void prolong_rows<float>(int, int, const float*, float*, hipStream_t);

// dst rows = src rows (widened to FP64) for the active problems, zero for the
// inactive ones
template <typename TS>
__global__ void k_copy_active_rows(long long per, int rows, int row0, const CgScal* scal,
                                   const TS* __restrict__ src, double* __restrict__ dst) {
  const long long total = per * rows;
  for (long long i = (long long)blockIdx.x * blockDim.x + threadIdx.x; i < total;
       i += (long long)gridDim.x * blockDim.x) {
    const int row = (int)(i / per);
    dst[i] = scal[row0 + row].active ? (double)src[i] : 0.0;
  }
}
template <typename TS>
void copy_active_rows(int n, int rows, int row0, const CgScal* scal, const TS* src, double* dst,
                      hipStream_t s) {
  if (rows <= 0) return;
  const long long per = (long long)lay_row(n);
  hipLaunchKernelGGL(k_copy_active_rows<TS>, dim3(grid_for(per * rows, 256)), dim3(256), 0, s,
                     per, rows, row0, scal, src, dst);
}
template void copy_active_rows<double>(int, int, int, const CgScal*, const double*, double*,
                                       hipStream_t);
template void copy_active_rows<float>(int, int, int, const CgScal*, const float*, double*,
                                      hipStream_t);
template void restrict_rows<double>(int, int, int, const CgScal*, const double*, double*,
                                    hipStream_t);
template void restrict_rows<float>(int, int, int, const CgScal*, const float*, float*,
                                   hipStream_t);
template void prolong_add_rows<double>(int, int, int, const CgScal*, const double*, double*,
                                       hipStream_t);
template void prolong_add_rows<float>(int, int, int, const CgScal*, const float*, float*,
                                      hipStream_t);

// ---------------------------------------------------------------------------
// Dense coarsest-grid solve.  A hierarchy whose top grid is n = 2^a b + 1
// with odd b > 1 cannot coarsen below b + 1 vertices per axis; that grid
// keeps (b - 1)^3 interior unknowns (at most 7^3 here) and is solved exactly
// with the inverse of its rediscretised operator, built per problem from the
// KL draw and applied as a small dense product in every V-cycle.
//
// The inverse comes from a blocked Cholesky factorisation A = L L^T on 16 x 16
// tiles.  Every tile product runs on the FP64 matrix cores
// (v_mfma_f64_16x16x4f64: four instructions per 16 x 16 x 16 product); the
// 16 x 16 diagonal blocks are factored and inverted on the vector ALUs in
// LDS.  Then W = L^-1 by blocked forward substitution, and A^-1 = W^T W.  The
// matrix is padded to Np = 16 ceil(N / 16) with the identity, whose inverse
// block is the identity again and is never read.  One workgroup of four waves
// per problem; A, then A^-1, lives in the problem's Np x Np block of `ainv`,
// W in the same block of `work` (both stay cache-resident at these sizes).
//
// MFMA operand layout (16 x 16 x 4, FP64): lane l supplies a = X[l % 16][k0 +
// l / 16] of the left factor and b = Y[k0 + l / 16][l % 16] of the right one,
// and holds C[4 r + l / 16][l % 16] in accumulator element r.
// ---------------------------------------------------------------------------
constexpr int DENSE_NMAX = 9;
constexpr int DT = 16;                 // tile edge
typedef double dbl4 __attribute__((ext_vector_type(4)));

__device__ __forceinline__ dbl4 mfma_f64(double a, double b, dbl4 c) {
  return __builtin_amdgcn_mfma_f64_16x16x4f64(a, b, c, 0, 0, 0);
}

// One wave's 16 x 16 tile of a row-major matrix with pitch ld at tile (I, J).
struct TileRef {
  double* m;
  int ld;
  __device__ double* at(int I, int J) const { return m + ((size_t)I * DT) * ld + (size_t)J * DT; }
};

__device__ __forceinline__ dbl4 tile_load_c(const double* t, int ld, int li, int lk) {
  dbl4 c;
#pragma unroll
  for (int r = 0; r < 4; ++r) c[r] = t[(4 * r + lk) * ld + li];
  return c;
}
__device__ __forceinline__ void tile_store_c(double* t, int ld, int li, int lk, dbl4 c) {
#pragma unroll
  for (int r = 0; r < 4; ++r) t[(4 * r + lk) * ld + li] = c[r];
}
// c += sign * X Y^T (X, Y tiles, row-major, pitch ld)
__device__ __forceinline__ dbl4 mma_xyt(const double* x, const double* y, int ld, int li, int lk,
                                        double sign, dbl4 c) {
#pragma unroll
  for (int sl = 0; sl < 4; ++sl)
    c = mfma_f64(sign * x[li * ld + 4 * sl + lk], y[li * ld + 4 * sl + lk], c);
  return c;
}
// c += sign * X Y
__device__ __forceinline__ dbl4 mma_xy(const double* x, int ldx, const double* y, int ldy, int li,
                                       int lk, double sign, dbl4 c) {
#pragma unroll
  for (int sl = 0; sl < 4; ++sl)
    c = mfma_f64(sign * x[li * ldx + 4 * sl + lk], y[(4 * sl + lk) * ldy + li], c);
  return c;
}
// c += X^T Y
__device__ __forceinline__ dbl4 mma_xty(const double* x, const double* y, int ld, int li, int lk,
                                        dbl4 c) {
#pragma unroll
  for (int sl = 0; sl < 4; ++sl)
    c = mfma_f64(x[(4 * sl + lk) * ld + li], y[(4 * sl + lk) * ld + li], c);
  return c;
}

__global__ void __launch_bounds__(256)
    k_dense_coarse_inv(int n, const double* __restrict__ coef, int K,
                       const double* __restrict__ cosT, double* __restrict__ ainv,
                       double* __restrict__ work) {
  __shared__ double sb[DENSE_NMAX * DENSE_NMAX * DENSE_NMAX];
  __shared__ double sc[KMAX * KMAX * KMAX];
  __shared__ double sd[DT][DT + 1];     // diagonal tile being factored (L)
  __shared__ double st[DT][DT + 1];     // its inverse T = L^-1
  __shared__ double sw[4][DT][DT + 1];  // one scratch tile per wave
  const int prob = blockIdx.x, tid = threadIdx.x;
  const int lane = tid & 63, wave = tid >> 6, li = lane & 15, lk = lane >> 4;
  const int m = n - 2, N = m * m * m, K3 = K * K * K;
  const int Np = (N + DT - 1) / DT * DT, nt = Np / DT;
  const TileRef A{ainv + (size_t)prob * Np * Np, Np};
  const TileRef W{work + (size_t)prob * Np * Np, Np};

  // the operator: 1/a at every vertex from the KL sum, harmonic faces
  for (int j = tid; j < K3; j += 256) sc[j] = coef[(size_t)prob * K3 + j];
  __syncthreads();
  for (int v = tid; v < n * n * n; v += 256) {
    const int ix = v / (n * n), iy = (v / n) % n, iz = v % n;
    double l = 0.0;
    for (int k1 = 0; k1 < K; ++k1)
      for (int k2 = 0; k2 < K; ++k2)
        for (int k3 = 0; k3 < K; ++k3)
          l += sc[(k1 * K + k2) * K + k3] * cosT[k1 * n + ix] * cosT[k2 * n + iy] *
               cosT[k3 * n + iz];
    sb[v] = exp(-l);
  }
  for (size_t e = tid; e < (size_t)Np * Np; e += 256) {
    const int i = (int)(e / Np), j = (int)(e % Np);
    A.m[e] = (i == j && i >= N) ? 1.0 : 0.0;
    W.m[e] = 0.0;
  }
  __syncthreads();
  const double ih2 = (double)(n - 1) * (double)(n - 1);
  for (int i = tid; i < N; i += 256) {
    const int ix = 1 + i / (m * m), iy = 1 + (i / m) % m, iz = 1 + i % m;
    const int v = (ix * n + iy) * n + iz;
    const int d[6][3] = {{-1, 0, 0}, {1, 0, 0}, {0, -1, 0}, {0, 1, 0}, {0, 0, -1}, {0, 0, 1}};
    double diag = 0.0;
    for (int f = 0; f < 6; ++f) {
      const int jx = ix + d[f][0], jy = iy + d[f][1], jz = iz + d[f][2];
      const double af = ih2 * face(sb[v], sb[(jx * n + jy) * n + jz]);
      diag += af;
      if (jx >= 1 && jx <= m && jy >= 1 && jy <= m && jz >= 1 && jz <= m)
        A.m[(size_t)i * Np + ((jx - 1) * m + (jy - 1)) * m + (jz - 1)] = -af;
    }
    A.m[(size_t)i * Np + i] = diag;
  }
  __syncthreads();

  // Cholesky, right-looking over tile columns k
  const int ti = tid / DT, tj = tid % DT;   // this thread's element of a 16 x 16 tile
  for (int k = 0; k < nt; ++k) {
    sd[ti][tj] = *(A.at(k, k) + ti * Np + tj);
    st[ti][tj] = 0.0;
    __syncthreads();
    for (int j = 0; j < DT; ++j) {           // unblocked factor of the diagonal tile
      if (ti == j && tj == j) sd[j][j] = sqrt(sd[j][j]);
      __syncthreads();
      if (tj == j && ti > j) sd[ti][j] /= sd[j][j];
      __syncthreads();
      if (tj > j && ti >= tj) sd[ti][tj] -= sd[ti][j] * sd[tj][j];
      __syncthreads();
    }
    for (int i = 0; i < DT; ++i) {           // T = L^-1, row by row
      if (ti == i && tj <= i) {
        double acc = (tj == i) ? 1.0 : 0.0;
        for (int q = tj; q < i; ++q) acc -= sd[i][q] * st[q][tj];
        st[i][tj] = acc / sd[i][i];
      }
      __syncthreads();
    }
    *(A.at(k, k) + ti * Np + tj) = tj <= ti ? sd[ti][tj] : 0.0;
    *(W.at(k, k) + ti * Np + tj) = st[ti][tj];
    // panel: L_ik = A_ik T^T, one tile per wave in turn
    for (int i = k + 1 + wave; i < nt; i += 4) {
      double* t = A.at(i, k);
      dbl4 c = {0.0, 0.0, 0.0, 0.0};
#pragma unroll
      for (int sl = 0; sl < 4; ++sl)
        c = mfma_f64(t[li * Np + 4 * sl + lk], st[li][4 * sl + lk], c);
      tile_store_c(t, Np, li, lk, c);
    }
    __syncthreads();
    // trailing update of the lower tiles: A_ij -= L_ik L_jk^T, k < j <= i
    const int rem = nt - 1 - k;
    for (int p = wave; p < rem * (rem + 1) / 2; p += 4) {
      int i = 0;
      while ((i + 1) * (i + 2) / 2 <= p) ++i;
      const int j = p - i * (i + 1) / 2;
      const int I = k + 1 + i, J = k + 1 + j;
      double* t = A.at(I, J);
      dbl4 c = tile_load_c(t, Np, li, lk);
      c = mma_xyt(A.at(I, k), A.at(J, k), Np, li, lk, -1.0, c);
      tile_store_c(t, Np, li, lk, c);
    }
    __syncthreads();
  }

  // W = L^-1: column blocks k in turn per wave; W_kk = T_k is already there,
  // W_ik = -T_i (sum_{k <= j < i} L_ij W_jk) for i > k
  for (int k = wave; k < nt; k += 4) {
    for (int i = k + 1; i < nt; ++i) {
      dbl4 c = {0.0, 0.0, 0.0, 0.0};
      for (int j = k; j < i; ++j) c = mma_xy(A.at(i, j), Np, W.at(j, k), Np, li, lk, 1.0, c);
#pragma unroll
      for (int r = 0; r < 4; ++r) sw[wave][4 * r + lk][li] = c[r];
      __builtin_amdgcn_fence(__ATOMIC_RELEASE, "wavefront");
      __builtin_amdgcn_wave_barrier();
      __builtin_amdgcn_fence(__ATOMIC_ACQUIRE, "wavefront");
      const double* Ti = W.at(i, i);
      dbl4 w = {0.0, 0.0, 0.0, 0.0};
#pragma unroll
      for (int sl = 0; sl < 4; ++sl)
        w = mfma_f64(-Ti[li * Np + 4 * sl + lk], sw[wave][4 * sl + lk][li], w);
      __builtin_amdgcn_fence(__ATOMIC_RELEASE, "wavefront");
      __builtin_amdgcn_wave_barrier();
      __builtin_amdgcn_fence(__ATOMIC_ACQUIRE, "wavefront");
      tile_store_c(W.at(i, k), Np, li, lk, w);
      // the tile is read back by other lanes of this wave for the next i
      __builtin_amdgcn_fence(__ATOMIC_RELEASE, "workgroup");
      __builtin_amdgcn_wave_barrier();
      __builtin_amdgcn_fence(__ATOMIC_ACQUIRE, "workgroup");
    }
  }
  __syncthreads();

  // A^-1 = W^T W: tile (I, J), I >= J, sum over K >= I of W_KI^T W_KJ,
  // written with its mirror (J, I) over the no longer needed factor
  for (int p = wave; p < nt * (nt + 1) / 2; p += 4) {
    int I = 0;
    while ((I + 1) * (I + 2) / 2 <= p) ++I;
    const int J = p - I * (I + 1) / 2;
    dbl4 c = {0.0, 0.0, 0.0, 0.0};
    for (int Kt = I; Kt < nt; ++Kt) c = mma_xty(W.at(Kt, I), W.at(Kt, J), Np, li, lk, c);
    tile_store_c(A.at(I, J), Np, li, lk, c);
    if (I != J) {
      double* t = A.at(J, I);
#pragma unroll
      for (int r = 0; r < 4; ++r) t[li * Np + 4 * r + lk] = c[r];
    }
  }
}

void dense_coarse_inv(int n, int rows, const double* coef, int K, const double* cosT,
                      double* ainv, double* work, hipStream_t s) {
  if (rows <= 0) return;
  hipLaunchKernelGGL(k_dense_coarse_inv, dim3(rows), dim3(256), 0, s, n, coef, K, cosT, ainv,
                     work);
}

// x = A^-1 b on the interior of every active problem's coarsest row (the
// inverse is symmetric, so thread i walks column i: coalesced reads).
template <typename T>
__global__ void __launch_bounds__(256)
    k_dense_apply(int n, const CgScal* __restrict__ scal, const double* __restrict__ ainv,
                  const T* __restrict__ b, T* __restrict__ x) {
  __shared__ double sbv[(DENSE_NMAX - 2) * (DENSE_NMAX - 2) * (DENSE_NMAX - 2)];
  const int prob = blockIdx.x, tid = threadIdx.x;
  if (scal && !scal[prob].active) return;  // uniform per workgroup
  const int m = n - 2, N = m * m * m;
  const size_t base = (size_t)prob * (size_t)lay_row(n);
  const int lp = lay_pitch(n), lo = lay_off(n);
  auto vtx = [&](int i) {
    return ((1 + i / (m * m)) * n + 1 + (i / m) % m) * lp + 1 + i % m + lo;
  };
  for (int i = tid; i < N; i += 256) sbv[i] = (double)b[base + vtx(i)];
  __syncthreads();
  const int Np = dense_pitch(N);
  const double* A = ainv + (size_t)prob * Np * Np;
  for (int i = tid; i < N; i += 256) {
    double acc = 0.0;
    for (int j = 0; j < N; ++j) acc += A[(size_t)j * Np + i] * sbv[j];
    x[base + vtx(i)] = (T)acc;
  }
}

template <typename T>
void dense_apply(int n, int rows, const CgScal* scal, const double* ainv, const T* b, T* x,
                 hipStream_t s) {
  if (rows <= 0) return;
  hipLaunchKernelGGL(k_dense_apply<T>, dim3(rows), dim3(256), 0, s, n, scal, ainv, b, x);
}
template void dense_apply<double>(int, int, const CgScal*, const double*, const double*, double*,
                                  hipStream_t);
template void dense_apply<float>(int, int, const CgScal*, const double*, const float*, float*,
                                 hipStream_t);

// Solver rows [count] written as dense [n][n][n] rows, row r at dst + dst_off[r]
// (dst_off null: row r at r n^3).
__global__ void k_unpack_rows(int n, int count, const long long* __restrict__ dst_off,
                              const double* __restrict__ src, double* __restrict__ dst) {
  const long long per = (long long)n * n * n, total = per * count;
  const long long srow = lay_row(n);
  const int lp = lay_pitch(n), lo = lay_off(n);
  for (long long e = (long long)blockIdx.x * blockDim.x + threadIdx.x; e < total;
       e += (long long)gridDim.x * blockDim.x) {
    const long long r = e / per, v = e - r * per;
    const long long xy = v / n;
    const int iz = (int)(v - xy * n);
    dst[(dst_off ? dst_off[r] : r * per) + v] = src[r * srow + xy * lp + iz + lo];
  }
}
void scatter_rows(int n, int count, const long long* dst_off, const double* src, double* dst,
                  hipStream_t s) {
  const long long total = (long long)n * n * n * count;
  if (total <= 0) return;
  hipLaunchKernelGGL(k_unpack_rows, dim3(grid_for(total, 256)), dim3(256), 0, s, n, count,
                     dst_off, src, dst);
}
void unpack_rows(int n, int rows, const double* src, double* dst, hipStream_t s) {
  scatter_rows(n, rows, nullptr, src, dst, s);
}

// Constant on the interior, zero on the boundary.
__global__ void k_fill_interior(int n, double v, double* __restrict__ out) {
  const long long N = (long long)n * n * n;
  for (long long e = (long long)blockIdx.x * blockDim.x + threadIdx.x; e < N;
       e += (long long)gridDim.x * blockDim.x) {
    const int ix = (int)(e / ((long long)n * n)), iy = (int)((e / n) % n), iz = (int)(e % n);
    out[e] = (ix > 0 && iy > 0 && iz > 0 && ix < n - 1 && iy < n - 1 && iz < n - 1) ? v : 0.0;
  }
}
void fill_interior(int n, double v, double* out, hipStream_t s) {
  hipLaunchKernelGGL(k_fill_interior, dim3(grid_for((long long)n * n * n, 256)), dim3(256), 0, s,
                     n, v, out);
}

// ---------------------------------------------------------------------------
// Random field: Philox4x64-10 (Salmon, Moraes, Dror, Shaw, SC'11) keyed by
// (seed, 0) with counter (block, sample, level, tag); Box-Muller normals; KL
// coefficients c_j = sqrt(sigma2 lam_k) xi_j, lam_k = (1 + |k|^2)^(-5/2).
// ---------------------------------------------------------------------------
__device__ __forceinline__ void philox_block(uint64_t c0, uint64_t c1, uint64_t c2, uint64_t c3,
                                             uint64_t k0, uint64_t k1, uint64_t w[4]) {
  const uint64_t M0 = 0xD2E7470EE14C6C93ULL, M1 = 0xCA5A826395121157ULL;
  const uint64_t W0 = 0x9E3779B97F4A7C15ULL, W1 = 0xBB67AE8584CAA73BULL;
#pragma unroll
  for (int rd = 0; rd < 10; ++rd) {
    if (rd > 0) {
      k0 += W0;
      k1 += W1;
    }
    const uint64_t lo0 = M0 * c0, hi0 = __umul64hi(M0, c0);
    const uint64_t lo1 = M1 * c2, hi1 = __umul64hi(M1, c2);
    const uint64_t n0 = hi1 ^ c1 ^ k0;
    const uint64_t n2 = hi0 ^ c3 ^ k1;
    c0 = n0;
    c1 = lo1;
    c2 = n2;
    c3 = lo0;
  }
  w[0] = c0; w[1] = c1; w[2] = c2; w[3] = c3;
}

__device__ __forceinline__ void normals4(uint64_t seed, int level, int64_t sample, int tag,
                                         int blk, double z[4]) {
  uint64_t w[4];
  philox_block((uint64_t)blk, (uint64_t)sample, (uint64_t)level, (uint64_t)tag, seed, 0ULL, w);
  const double two_pi = 2.0 * 3.14159265358979323846;
#pragma unroll
  for (int pr = 0; pr < 2; ++pr) {
    const double u1 = ((double)(w[2 * pr] >> 11) + 0.5) * 0x1.0p-53;
    const double u2 = ((double)(w[2 * pr + 1] >> 11) + 0.5) * 0x1.0p-53;
    const double r = sqrt(-2.0 * log(u1));
    const double t = two_pi * u2;
    z[2 * pr] = r * cos(t);
    z[2 * pr + 1] = r * sin(t);
  }
}

// Four draws of block blk in draw order: law 0 standard normals (Box-Muller),
// law 1 uniforms on (-4, 4) (xi = -4 + 8 u of the same 53-bit uniforms).
__device__ __forceinline__ void draws4(uint64_t seed, int level, int64_t sample, int blk,
                                       int law, double z[4]) {
  if (law == 0) {
    normals4(seed, level, sample, 0, blk, z);
    return;
  }
  uint64_t w[4];
  philox_block((uint64_t)blk, (uint64_t)sample, (uint64_t)level, 0ULL, seed, 0ULL, w);
#pragma unroll
  for (int q = 0; q < 4; ++q) z[q] = -4.0 + 8.0 * (((double)(w[q] >> 11) + 0.5) * 0x1.0p-53);
}

// KL coefficient of draw t, stored at its evaluation index (k1, k2, k3) <->
// cos(k1 pi x) cos(k2 pi y) cos(k3 pi z), e = ((k1-1) K + (k2-1)) K + (k3-1).
// law 0: t = e, lam = (1 + |k|^2)^(-5/2).
// law 1 (Sec. 5): draw t = ((j-1) K + (k-1)) K + (l-1) multiplies
// cos(j pi y) cos(k pi z) cos(l pi x), so it lands at (k1, k2, k3) = (l, j, k);
// lam = exp(-pi (j + k + l) rho).
__device__ __forceinline__ void kl_term(int t, int K, int law, double rho, int* e, double* lam) {
  const int a = t / (K * K) + 1, b = (t / K) % K + 1, c = t % K + 1;
  if (law == 0) {
    *e = t;
    *lam = pow(1.0 + (double)(a * a + b * b + c * c), -2.5);
  } else {
    *e = ((c - 1) * K + (a - 1)) * K + (b - 1);
    *lam = exp(-3.14159265358979323846 * (double)(a + b + c) * rho);
  }
}

__global__ void k_kl_coeffs(const int* __restrict__ prob_level,
                            const int64_t* __restrict__ prob_sample, int nprob, uint64_t seed,
                            int K, double sigma2, int law, double rho,
                            double* __restrict__ coef) {
  const int K3 = K * K * K;
  const int nblk = (K3 + 3) / 4;
  const long long total = (long long)nprob * nblk;
  for (long long i = (long long)blockIdx.x * blockDim.x + threadIdx.x; i < total;
       i += (long long)gridDim.x * blockDim.x) {
    const int p = (int)(i / nblk), b = (int)(i % nblk);
    double z[4];
    draws4(seed, prob_level[p], prob_sample[p], b, law, z);
    for (int q = 0; q < 4; ++q) {
      const int t = 4 * b + q;
      if (t >= K3) break;
      int e;
      double lam;
      kl_term(t, K, law, rho, &e, &lam);
      coef[(size_t)p * K3 + e] = sqrt(sigma2) * sqrt(lam) * z[q];
    }
  }
}
__global__ void k_kl_draws(uint64_t seed, int level, int64_t first, int64_t count, int K3,
                           int law, double* __restrict__ xi) {
  const int nblk = (K3 + 3) / 4;
  const long long total = count * nblk;
  for (long long i = (long long)blockIdx.x * blockDim.x + threadIdx.x; i < total;
       i += (long long)gridDim.x * blockDim.x) {
    const long long m = i / nblk;
    const int b = (int)(i % nblk);
    double z[4];
    draws4(seed, level, first + m, b, law, z);
    for (int q = 0; q < 4; ++q) {
      const int j = 4 * b + q;
      if (j < K3) xi[m * K3 + j] = z[q];
    }
  }
}

__global__ void k_philox_words(uint64_t seed, int level, int64_t sample, int tag, int nblocks,
                               uint64_t* out) {
  const int b = blockIdx.x * blockDim.x + threadIdx.x;
  if (b >= nblocks) return;
  uint64_t w[4];
  philox_block((uint64_t)b, (uint64_t)sample, (uint64_t)level, (uint64_t)tag, seed, 0ULL, w);
  for (int q = 0; q < 4; ++q) out[4 * b + q] = w[q];
}

__global__ void k_cos_table(int n, int K, double* out) {
  const int i = blockIdx.x * blockDim.x + threadIdx.x;
  if (i >= n * K) return;
  const int k = i / n + 1, v = i % n;
  const double h = 1.0 / (double)(n - 1);
  out[i] = cos(3.14159265358979323846 * (double)k * ((double)v * h));
}

void kl_coeffs(const int* prob_level, const int64_t* prob_sample, int nprob, uint64_t seed,
               int K, double sigma2, int law, double rho, double* coef, hipStream_t s) {
  if (nprob <= 0) return;
  const long long total = (long long)nprob * ((K * K * K + 3) / 4);
  hipLaunchKernelGGL(k_kl_coeffs, dim3(grid_for(total, 256)), dim3(256), 0, s, prob_level,
                     prob_sample, nprob, seed, K, sigma2, law, rho, coef);
}
void kl_draws(uint64_t seed, int level, int64_t first, int64_t count, int K3, int law,
              double* xi, hipStream_t s) {
  if (count <= 0) return;
  const long long total = count * ((K3 + 3) / 4);
  hipLaunchKernelGGL(k_kl_draws, dim3(grid_for(total, 256)), dim3(256), 0, s, seed, level,
                     first, count, K3, law, xi);
}
void philox_words(uint64_t seed, int level, int64_t sample, int tag, int nblocks, uint64_t* out,
                  hipStream_t s) {
  if (nblocks <= 0) return;
  hipLaunchKernelGGL(k_philox_words, dim3(cdiv(nblocks, 64)), dim3(64), 0, s, seed, level,
                     sample, tag, nblocks, out);
}
void cos_table(int n, int K, double* out, hipStream_t s) {
  hipLaunchKernelGGL(k_cos_table, dim3(cdiv((long long)n * K, 256)), dim3(256), 0, s, n, K, out);
}

// ---------------------------------------------------------------------------
// Elementwise kernels over the rows of one group.  A row is cut into
// tiles_per_row contiguous chunks, one workgroup each, so partial sums land
// in fixed slots and every reduction is deterministic.
// ---------------------------------------------------------------------------
// dense field src copied into every solver row of dst (padding untouched)
__global__ void k_rows_broadcast(int n, long long total, const double* __restrict__ src,
                                 double* __restrict__ dst) {
  const long long per = (long long)n * n * n, drow = lay_row(n);
  const int lp = lay_pitch(n), lo = lay_off(n);
  for (long long e = (long long)blockIdx.x * blockDim.x + threadIdx.x; e < total;
       e += (long long)gridDim.x * blockDim.x) {
    const long long r = e / per, v = e - r * per;
    const long long xy = v / n;
    const int iz = (int)(v - xy * n);
    dst[r * drow + xy * lp + iz + lo] = src[v];
  }
}
void rows_broadcast(int n, int rows, const double* src, double* dst, hipStream_t s) {
  const long long total = (long long)n * n * n * rows;
  if (total <= 0) return;
  hipLaunchKernelGGL(k_rows_broadcast, dim3(grid_for(total, 256)), dim3(256), 0, s, n, total,
                     src, dst);
}
__global__ void k_to_f32(long long count, const double* __restrict__ x, float* __restrict__ y) {
  for (long long i = (long long)blockIdx.x * blockDim.x + threadIdx.x; i < count;
       i += (long long)gridDim.x * blockDim.x)
    y[i] = (float)x[i];
}
void to_f32(long long count, const double* x, float* y, hipStream_t s) {
  if (count <= 0) return;
  hipLaunchKernelGGL(k_to_f32, dim3(grid_for(count, 256)), dim3(256), 0, s, count, x, y);
}
__global__ void k_zero(long long count, double* x) {
  for (long long i = (long long)blockIdx.x * blockDim.x + threadIdx.x; i < count;
       i += (long long)gridDim.x * blockDim.x)
    x[i] = 0.0;
}
void rows_zero(long long count, double* x, hipStream_t s) {
  if (count <= 0) return;
  hipLaunchKernelGGL(k_zero, dim3(grid_for(count, 256)), dim3(256), 0, s, count, x);
}

enum GroupOp { G_DOT = 0, G_UPDATE = 1, G_MISFIT = 2, G_RUPDATE = 3, G_XFLUSH = 4 };

// Elementwise step of one group op at solver-row element k (interior vertex
// (ix, iy, iz)); returns the term of the workgroup's partial sum.
template <int OP>
__device__ __forceinline__ double group_elem(size_t k, int n, int ix, int iy, int iz, double al,
                                             double* __restrict__ a, const double* __restrict__ b,
                                             double* __restrict__ c,
                                             const double* __restrict__ d,
                                             float* __restrict__ cf) {
  if (OP == G_DOT) return a[k] * b[k];
  if (OP == G_XFLUSH) {
    a[k] = a[k] + al * b[k];
    return 0.0;
  }
  if (OP == G_UPDATE || OP == G_RUPDATE) {
    if (OP == G_UPDATE) a[k] = a[k] + al * b[k];
    const double r = c[k] - al * d[k];
    c[k] = r;
    if (cf) cf[k] = (float)r;
    return r * r;
  }
  // G_MISFIT
  const double r = a[k] - b[((size_t)ix * n + iy) * n + iz];
  c[k] = r;
  a[k] = 0.0;
  return r * r;
}

// Group ops over the rows of one group; each row is cut into tiles_per_row
// workgroups whose partial sums land in fixed slots (deterministic sums).
//   G_DOT    : <a, b>
//   G_UPDATE : a += alpha b (x += alpha p), c -= alpha d (r -= alpha q),
//              <c, c>; cf (nullable) receives c in FP32
//   G_RUPDATE: G_UPDATE without a (the matvec applies x's step one
//              iteration later)
//   G_XFLUSH : a += alpha b, b being d where the scalars say the pending
//              step's direction is in the second buffer; every problem with
//              a pending step, active or not; no partial sums
//   G_MISFIT : c = a - y_d (b: dense y_d, shared), a = 0, <c, c>
// Only interior vertices are visited: boundary vertices and padding of these
// rows hold zeros that every op leaves unchanged.  On grids of 65 and more
// vertices a wave walks whole interior z lines (z = 1 .. n-2, 64 lanes
// abreast), skipping the boundary planes, lines and padding in memory.  NZ > 0
// is the number of 64-point chunks of a line (n - 1 <= 64 NZ): a lane then
// handles LU = max(1, 4 / NZ) lines per step and issues the loads of all its
// LU x NZ points before any store.  These lines also take the boundary
// vertex z = n - 1 (a zero in every operand, so unchanged): with the padded
// layout the stores then cover whole 128-byte lines.  NZ = 0 walks lines of any length one
// chunk at a time; NZ = -1 (grids below 65) strides over the dense row: the
// misfit tests each vertex, the dot and the update stream every element
// (boundary zeros pass through unchanged), four per thread in flight.
template <int OP, int NZ>
__device__ __forceinline__ void group_tile(const GridArgs& g, int bid, double* sred,
                                           double* __restrict__ a, const double* __restrict__ b,
                                           double* __restrict__ c, const double* __restrict__ d,
                                           const int* __restrict__ poff,
                                           double* __restrict__ partial,
                                           float* __restrict__ cf) {
  const int tpr = g.t.tiles_per_row;
  const int row = bid / tpr;
  const int tile = bid - row * tpr;
  const int prob = g.row0 + row;
  if (OP == G_XFLUSH) {
    if (!g.scal[prob].pending) return;  // uniform per workgroup
  } else if (g.scal && !g.scal[prob].active) {
    return;
  }
  const int n = g.n, m = n - 2;
  const size_t base = (size_t)row * (size_t)g.stride;
  constexpr bool STEP = OP == G_UPDATE || OP == G_RUPDATE || OP == G_XFLUSH;
  constexpr bool LOAD_AB = OP == G_DOT || OP == G_UPDATE || OP == G_XFLUSH;
  constexpr bool LOAD_CD = OP == G_UPDATE || OP == G_RUPDATE;
  const double al = STEP ? g.scal[prob].alpha : 0.0;
  if (OP == G_XFLUSH && g.scal[prob].pbuf) b = d;
  double acc = 0.0;
  if constexpr (NZ >= 0) {
    const int lp = lay_pitch(n), lo = lay_off(n);
    const long long lines = (long long)m * m;
    const long long per = (lines + tpr - 1) / tpr;
    const long long l0 = (long long)tile * per, l1 = min(lines, l0 + per);
    const int wave = threadIdx.x >> 6, lane = threadIdx.x & 63;
    if constexpr (NZ > 0 && OP != G_MISFIT) {
      constexpr int LU = NZ >= 4 ? 1 : 4 / NZ;
      for (long long l = l0 + wave; l < l1; l += 4 * LU) {
        size_t k[LU][NZ];
        bool ok[LU][NZ];
        double va[LU][NZ], vb[LU][NZ], vc[LU][NZ], vd[LU][NZ];
#pragma unroll
        for (int u = 0; u < LU; ++u) {
          const long long ll = l + 4 * u;
          const int ix = 1 + (int)(ll / m), iy = 1 + (int)(ll % m);
          const size_t lb = base + ((size_t)ix * n + iy) * lp + lo;
#pragma unroll
          for (int j = 0; j < NZ; ++j) {
            const int iz = 1 + lane + 64 * j;
            ok[u][j] = ll < l1 && iz <= m + 1;
            k[u][j] = lb + iz;
            if (ok[u][j]) {
              if (LOAD_AB) {
                va[u][j] = a[k[u][j]];
                vb[u][j] = b[k[u][j]];
              }
              if (LOAD_CD) {
                vc[u][j] = c[k[u][j]];
                vd[u][j] = d[k[u][j]];
              }
            }
          }
        }
#pragma unroll
        for (int u = 0; u < LU; ++u) {
#pragma unroll
          for (int j = 0; j < NZ; ++j) {
            if (!ok[u][j]) continue;
            if (OP == G_DOT) {
              acc += va[u][j] * vb[u][j];
            } else if (OP == G_XFLUSH) {
              a[k[u][j]] = va[u][j] + al * vb[u][j];
            } else {
              if (OP == G_UPDATE) a[k[u][j]] = va[u][j] + al * vb[u][j];
              const double r = vc[u][j] - al * vd[u][j];
              c[k[u][j]] = r;
              if (cf) cf[k[u][j]] = (float)r;
              acc += r * r;
            }
          }
        }
      }
    } else {
      for (long long l = l0 + wave; l < l1; l += 4) {
        const int ix = 1 + (int)(l / m), iy = 1 + (int)(l % m);
        const size_t lb = base + ((size_t)ix * n + iy) * lp + lo;
        for (int iz = 1 + lane; iz <= m; iz += 64)
          acc += group_elem<OP>(lb + iz, n, ix, iy, iz, al, a, b, c, d, cf);
      }
    }
  } else {
    const long long N = g.stride;
    const long long chunk = (N + tpr - 1) / tpr;
    const long long lo = (long long)tile * chunk;
    const long long hi = min(N, lo + chunk);
    long long i = lo + threadIdx.x;
    if (OP == G_MISFIT) {
      for (; i < hi; i += 256) {
        const int ix = (int)(i / ((long long)n * n)), iy = (int)((i / n) % n), iz = (int)(i % n);
        if (ix > 0 && iy > 0 && iz > 0 && ix < n - 1 && iy < n - 1 && iz < n - 1)
          acc += group_elem<OP>(base + i, n, ix, iy, iz, al, a, b, c, d, cf);
      }
    } else {
      constexpr int U = 4;
      for (; i + (U - 1) * 256 < hi; i += U * 256) {
        double va[U], vb[U], vc[U], vd[U];
#pragma unroll
        for (int u = 0; u < U; ++u) {
          const size_t k = base + i + u * 256;
          if (LOAD_AB) {
            va[u] = a[k];
            vb[u] = b[k];
          }
          if (LOAD_CD) {
            vc[u] = c[k];
            vd[u] = d[k];
          }
        }
#pragma unroll
        for (int u = 0; u < U; ++u) {
          const size_t k = base + i + u * 256;
          if (OP == G_DOT) {
            acc += va[u] * vb[u];
          } else if (OP == G_XFLUSH) {
            a[k] = va[u] + al * vb[u];
          } else {
            if (OP == G_UPDATE) a[k] = va[u] + al * vb[u];
            const double r = vc[u] - al * vd[u];
            c[k] = r;
            if (cf) cf[k] = (float)r;
            acc += r * r;
          }
        }
      }
      for (; i < hi; i += 256) acc += group_elem<OP>(base + i, n, 0, 0, 0, al, a, b, c, d, cf);
    }
  }
  if constexpr (OP != G_XFLUSH) {
    const double sum = block_sum<256>(acc, sred);
    if (threadIdx.x == 0) partial[poff[prob] + tile] = sum;
  }
}

template <int OP, int NZ>
__global__ void __launch_bounds__(256)
    k_group(GridArgs g, double* __restrict__ a, const double* __restrict__ b,
            double* __restrict__ c, const double* __restrict__ d, const int* __restrict__ poff,
            double* __restrict__ partial, float* __restrict__ cf) {
  __shared__ double sred[4];
  group_tile<OP, NZ>(g, blockIdx.x, sred, a, b, c, d, poff, partial, cf);
}

// The op over the rows of several groups in one launch (as k_march_groups).
template <int OP>
__global__ void __launch_bounds__(256)
    k_groups(GroupTable t, const int* __restrict__ poff, double* __restrict__ partial) {
  __shared__ double sred[4];
  int i = 0;
  while (i + 1 < t.count && (int)blockIdx.x >= t.gr[i + 1].begin) ++i;
  const GroupRows& r = t.gr[i];
  const int bid = (int)blockIdx.x - r.begin, m = r.g.n - 2;
  if (m < 63)
    group_tile<OP, -1>(r.g, bid, sred, r.a, r.b, r.c, r.d, poff, partial, r.cf);
  else if (m <= 64)
    group_tile<OP, 1>(r.g, bid, sred, r.a, r.b, r.c, r.d, poff, partial, r.cf);
  else if (m <= 128)
    group_tile<OP, 2>(r.g, bid, sred, r.a, r.b, r.c, r.d, poff, partial, r.cf);
  else if (m <= 256)
    group_tile<OP, 4>(r.g, bid, sred, r.a, r.b, r.c, r.d, poff, partial, r.cf);
  else
    group_tile<OP, 0>(r.g, bid, sred, r.a, r.b, r.c, r.d, poff, partial, r.cf);
}

template <int OP>
static void launch_group(const GridArgs& g, double* a, const double* b, double* c,
                         const double* d, const int* poff, double* partial, float* cf,
                         hipStream_t s) {
  if (g.rows <= 0) return;
  const dim3 grid(g.rows * g.t.tiles_per_row), block(256);
  const int m = g.n - 2;
  if (m < 63)
    hipLaunchKernelGGL((k_group<OP, -1>), grid, block, 0, s, g, a, b, c, d, poff, partial, cf);
  else if (m <= 64)
    hipLaunchKernelGGL((k_group<OP, 1>), grid, block, 0, s, g, a, b, c, d, poff, partial, cf);
  else if (m <= 128)
    hipLaunchKernelGGL((k_group<OP, 2>), grid, block, 0, s, g, a, b, c, d, poff, partial, cf);
  else if (m <= 256)
    hipLaunchKernelGGL((k_group<OP, 4>), grid, block, 0, s, g, a, b, c, d, poff, partial, cf);
  else
    hipLaunchKernelGGL((k_group<OP, 0>), grid, block, 0, s, g, a, b, c, d, poff, partial, cf);
}

template <int OP>
static void launch_groups(GroupTable& t, const int* poff, double* partial, hipStream_t s) {
  long long wg = 0;
  for (int i = 0; i < t.count; ++i) {
    t.gr[i].begin = (int)wg;
    wg += (long long)t.gr[i].g.rows * t.gr[i].g.t.tiles_per_row;
  }
  if (t.count == 1 || wg > MAX_WG256) {
    for (int i = 0; i < t.count; ++i) {
      const GroupRows& r = t.gr[i];
      launch_group<OP>(r.g, r.a, r.b, r.c, r.d, poff, partial, r.cf, s);
    }
    return;
  }
  if (wg > 0) hipLaunchKernelGGL((k_groups<OP>), dim3((unsigned)wg), dim3(256), 0, s, t, poff, partial);
}

void group_dot(const GridArgs& g, const double* a, const double* b, const int* poff,
               double* partial, hipStream_t s) {
  launch_group<G_DOT>(g, (double*)a, b, nullptr, nullptr, poff, partial, nullptr, s);
}
void group_update(const GridArgs& g, double* x, const double* p, double* r, const double* q,
                  const int* poff, double* partial, float* r32, hipStream_t s) {
  launch_group<G_UPDATE>(g, x, p, r, q, poff, partial, r32, s);
}
void group_misfit(const GridArgs& g, double* y, const double* yd, double* b_rows,
                  const int* poff, double* partial, hipStream_t s) {
  launch_group<G_MISFIT>(g, y, yd, b_rows, nullptr, poff, partial, nullptr, s);
}
void group_rupdate(GroupTable& t, const int* poff, double* partial, hipStream_t s) {
  launch_groups<G_RUPDATE>(t, poff, partial, s);
}
void group_xflush(GroupTable& t, hipStream_t s) { launch_groups<G_XFLUSH>(t, nullptr, nullptr, s); }

// ---------------------------------------------------------------------------
// Per-problem scalar steps (fixed summation order; the count of active problems
// an integer).
// ---------------------------------------------------------------------------
// LP lanes per problem sum its partial slots and the first of them takes the
// step.  The launch picks LP by the longest slot list: one thread alone walked
// the 1024 slots of a 257^3 problem in 31 us, a wave takes 5; problems of one
// slot (9^3) need no second lane.  The count of problems still active is
// gathered with integer atomics (exact, order-independent) into a counter that
// an earlier phase of the same iteration cleared (`clear`).
template <int LP>
__global__ void __launch_bounds__(256)
    k_cg_scalar(int phase, CgScal* scal, int nprob, const int* __restrict__ poff,
                const int* __restrict__ pcnt, const double* __restrict__ partial, double rtol,
                int max_iters, int* active_count, int aux, int* clear) {
  __shared__ int scount[4];
  int cnt = 0;
  const double rt2 = rtol * rtol;
  const int sub = threadIdx.x % LP;
  const int p = (blockIdx.x * 256 + threadIdx.x) / LP;
  if (p < nprob) {
    double sum = 0.0;
    if (partial) sum = slots_sum<LP>(partial + poff[p], pcnt[p], sub);
    if (sub == 0) {
    CgScal sc = scal[p];
    switch (phase) {
      case PH_INIT_BB:
        sc.bb = sum;
        sc.rr = sum;
        sc.active = sum > 0.0;
        sc.iters = 0;
        sc.alpha = 0.0;
        sc.beta = 0.0;
        sc.rz = 0.0;
        sc.pq = 0.0;
        sc.pending = 0;
        sc.pbuf = 0;
        sc.restart = 0;
        break;
      case PH_RZ0:
        if (sc.active) {
          sc.rz = sum;
          sc.beta = 0.0;
          sc.pending = 0;
        }
        break;
      case PH_RZ0_RR:
        if (sc.active) {
          sc.rz = sc.rr;
          sc.beta = 0.0;
          sc.pending = 0;
        }
        break;
      case PH_ALPHA:
        // the matvec just run applied the previous step of x; this one is
        // pending until the next matvec (or the flush before the residual
        // check) applies it from direction buffer aux
        if (sc.active) {
          sc.pq = sum;
          if (sum > 0.0) {
            sc.alpha = sc.rz / sum;
            sc.pending = 1;
            sc.pbuf = aux;
          } else {
            sc.alpha = 0.0;
            sc.active = 0;
            sc.pending = 0;
          }
        }
        break;
      case PH_RR:
        if (sc.active) {
          sc.rr = sum;
          sc.iters += 1;
          if (!(sum > rt2 * sc.bb) || sc.iters >= max_iters) sc.active = 0;
        }
        break;
      case PH_RZ:
        if (sc.active) {
          sc.beta = sum / sc.rz;
          sc.rz = sum;
        }
        break;
      case PH_RZ_RR:
        if (sc.active) {
          sc.beta = sc.rr / sc.rz;
          sc.rz = sc.rr;
        }
        break;
      case PH_TRUE:
        sc.rr = sum;
        sc.active = (sc.bb > 0.0) && (sum > rt2 * sc.bb) && (sc.iters < max_iters);
        sc.restart = sc.active;
        sc.alpha = 0.0;
        sc.beta = 0.0;
        sc.pending = 0;
        break;
      case PH_RECHECK:
        sc.active = sc.restart;
        break;
      case PH_FORCE_RESTART:
        if ((p & 1) == 0 && sc.bb > 0.0) {
          sc.active = 1;
          sc.restart = 1;
        }
        break;
    }
    scal[p] = sc;
    cnt = sc.active;
    }
  }
  if (clear && blockIdx.x == 0 && threadIdx.x == 0) *clear = 0;
  if (!active_count) return;   // uniform
  const unsigned long long on = __ballot(cnt != 0);
  if ((threadIdx.x & 63) == 0) scount[threadIdx.x >> 6] = __popcll(on);
  __syncthreads();
  if (threadIdx.x == 0) {
    const int c = scount[0] + scount[1] + scount[2] + scount[3];
    if (c) atomicAdd(active_count, c);
  }
}

__global__ void k_level_work_zero(EpiOut* out) {
  if (threadIdx.x < 8) out->work[threadIdx.x] = 0ull;
}
void level_work_zero(EpiOut* out, hipStream_t s) {
  hipLaunchKernelGGL(k_level_work_zero, dim3(1), dim3(64), 0, s, out);
}
// Integer sums (exact, order-independent) of the problems' interior unknowns
// x iterations per level.
__global__ void k_level_work_add(int count, unsigned long long per, const int* __restrict__ lvl,
                                 const CgScal* __restrict__ scal, EpiOut* out) {
  const int p = blockIdx.x * blockDim.x + threadIdx.x;
  if (p >= count) return;
  const int l = lvl[p];
  if (l >= 0 && l < 8) atomicAdd(&out->work[l], per * (unsigned long long)scal[p].iters);
}
void level_work_add(int count, int n, const int* prob_level, const CgScal* scal, EpiOut* out,
                    hipStream_t s) {
  if (count <= 0) return;
  const unsigned long long per = (unsigned long long)(n - 2) * (n - 2) * (n - 2);
  hipLaunchKernelGGL(k_level_work_add, dim3((count + 255) / 256), dim3(256), 0, s, count, per,
                     prob_level, scal, out);
}

// lanes that sum one problem's slots: one up to 4 slots, 8 up to 64, else a wave
static int slot_lanes(const double* partial, int max_slots) {
  return !partial || max_slots <= 4 ? 1 : max_slots <= 64 ? 8 : 64;
}

void cg_scalar(int phase, CgScal* scal, int nprob, int max_slots, const int* poff, const int* pcnt,
               const double* partial, double rtol, int max_iters, int* active_count, int* clear,
               hipStream_t s, int aux) {
  const int lp = slot_lanes(partial, max_slots);
#define MLSGD_LAUNCH(LP_)                                                                       \
  hipLaunchKernelGGL(k_cg_scalar<LP_>, dim3(cdiv((long long)nprob * LP_, 256)), dim3(256), 0, s, \
                     phase, scal, nprob, poff, pcnt, partial, rtol, max_iters, active_count, aux, \
                     clear)
  if (lp == 1)
    MLSGD_LAUNCH(1);
  else if (lp == 8)
    MLSGD_LAUNCH(8);
  else
    MLSGD_LAUNCH(64);
#undef MLSGD_LAUNCH
}

__global__ void __launch_bounds__(1024)
    k_scal_stats(const CgScal* scal, int nprob, double rtol, int* iters_max, int* nonconv,
                 double* relres_max) {
  __shared__ int si[1024], sn[1024];
  __shared__ double sr[1024];
  int it = 0, nc = 0;
  double rr = 0.0;
  for (int p = threadIdx.x; p < nprob; p += 1024) {
    const CgScal sc = scal[p];
    it = max(it, sc.iters);
    const double rel = sc.bb > 0.0 ? sqrt(sc.rr / sc.bb) : 0.0;
    if (!(rel <= rtol)) nc += 1;
    rr = fmax(rr, rel != rel ? 1e300 : rel);
  }
  si[threadIdx.x] = it;
  sn[threadIdx.x] = nc;
  sr[threadIdx.x] = rr;
  __syncthreads();
  for (int o = 512; o > 0; o >>= 1) {
    if (threadIdx.x < o) {
      si[threadIdx.x] = max(si[threadIdx.x], si[threadIdx.x + o]);
      sn[threadIdx.x] += sn[threadIdx.x + o];
      sr[threadIdx.x] = fmax(sr[threadIdx.x], sr[threadIdx.x + o]);
    }
    __syncthreads();
  }
  if (threadIdx.x == 0) {
    *iters_max = si[0];
    *nonconv = sn[0];
    *relres_max = sr[0];
  }
}
void scal_to_stats(const CgScal* scal, int nprob, double rtol, int* iters_max, int* nonconv,
                   double* relres_max, hipStream_t s) {
  hipLaunchKernelGGL(k_scal_stats, dim3(1), dim3(1024), 0, s, scal, nprob, rtol, iters_max,
                     nonconv, relres_max);
}

template <int LP>
__global__ void k_sum_partials(int nprob, const int* poff, const int* pcnt,
                               const double* partial, double scale, double* dst) {
  const int p = (blockIdx.x * blockDim.x + threadIdx.x) / LP;
  if (p >= nprob) return;
  const double sum = slots_sum<LP>(partial + poff[p], pcnt[p], threadIdx.x % LP);
  if (threadIdx.x % LP == 0) dst[p] = scale * sum;
}
void sum_partials(int nprob, int slots, const int* poff, const int* pcnt, const double* partial,
                  double scale, double* dst, hipStream_t s) {
  if (nprob <= 0) return;
  const int lp = slot_lanes(partial, slots);
#define MLSGD_LAUNCH(LP_)                                                                          \
  hipLaunchKernelGGL(k_sum_partials<LP_>, dim3(cdiv((long long)nprob * LP_, 256)), dim3(256), 0, s, \
                     nprob, poff, pcnt, partial, scale, dst)
  if (lp == 1)
    MLSGD_LAUNCH(1);
  else if (lp == 8)
    MLSGD_LAUNCH(8);
  else
    MLSGD_LAUNCH(64);
#undef MLSGD_LAUNCH
}

// ---------------------------------------------------------------------------
// Whole-field kernels on one grid.
// ---------------------------------------------------------------------------
__device__ __forceinline__ bool interior(int n, int ix, int iy, int iz) {
  return ix > 0 && iy > 0 && iz > 0 && ix < n - 1 && iy < n - 1 && iz < n - 1;
}

__global__ void k_restrict_full(int nf, const double* __restrict__ f, double* __restrict__ c) {
  const int nc = (nf - 1) / 2 + 1;
  const long long N = (long long)nc * nc * nc;
  for (long long i = (long long)blockIdx.x * blockDim.x + threadIdx.x; i < N;
       i += (long long)gridDim.x * blockDim.x) {
    const int jx = (int)(i / ((long long)nc * nc)), jy = (int)((i / nc) % nc), jz = (int)(i % nc);
    if (!interior(nc, jx, jy, jz)) {
      c[i] = 0.0;
      continue;
    }
    double acc = 0.0;
    for (int dx = -1; dx <= 1; ++dx) {
      const double wx = dx == 0 ? 0.5 : 0.25;
      double ay = 0.0;
      for (int dy = -1; dy <= 1; ++dy) {
        const double wy = dy == 0 ? 0.5 : 0.25;
        const double* p = f + ((size_t)(2 * jx + dx) * nf + (2 * jy + dy)) * nf + 2 * jz;
        ay += wy * (0.25 * p[-1] + 0.5 * p[0] + 0.25 * p[1]);
      }
      acc += wx * ay;
    }
    c[i] = acc;
  }
}
void restrict_full(int nf, const double* fine, double* coarse, hipStream_t s) {
  const int nc = (nf - 1) / 2 + 1;
  hipLaunchKernelGGL(k_restrict_full, dim3(grid_for((long long)nc * nc * nc, 256)), dim3(256), 0,
                     s, nf, fine, coarse);
}

// trilinear prolongation at fine vertex (ix, iy, iz) of the coarse field c
// stored with z pitch cp and offset co
__device__ __forceinline__ double prolong_at(int nc, int cp, int co, const double* __restrict__ c,
                                             int ix, int iy, int iz) {
  const int ax = ix >> 1, bx = (ix + 1) >> 1;
  const int ay = iy >> 1, by = (iy + 1) >> 1;
  const int az = iz >> 1, bz = (iz + 1) >> 1;
  auto cv = [&](int a, int b, int d) { return c[((size_t)a * nc + b) * cp + d + co]; };
  double v = cv(ax, ay, az);
  if (iz & 1) v += cv(ax, ay, bz);
  if (iy & 1) {
    v += cv(ax, by, az);
    if (iz & 1) v += cv(ax, by, bz);
  }
  if (ix & 1) {
    v += cv(bx, ay, az);
    if (iz & 1) v += cv(bx, ay, bz);
    if (iy & 1) {
      v += cv(bx, by, az);
      if (iz & 1) v += cv(bx, by, bz);
    }
  }
  const double w = ((ix & 1) ? 0.5 : 1.0) * ((iy & 1) ? 0.5 : 1.0) * ((iz & 1) ? 0.5 : 1.0);
  return w * v;
}

__global__ void k_prolong_full(int nc, const double* __restrict__ c, double* __restrict__ f) {
  const int nf = 2 * (nc - 1) + 1;
  const long long N = (long long)nf * nf * nf;
  for (long long i = (long long)blockIdx.x * blockDim.x + threadIdx.x; i < N;
       i += (long long)gridDim.x * blockDim.x) {
    const int ix = (int)(i / ((long long)nf * nf)), iy = (int)((i / nf) % nf), iz = (int)(i % nf);
    f[i] = interior(nf, ix, iy, iz) ? prolong_at(nc, nc, 0, c, ix, iy, iz) : 0.0;
  }
}
void prolong_full(int nc, const double* coarse, double* fine, hipStream_t s) {
  const int nf = 2 * (nc - 1) + 1;
  hipLaunchKernelGGL(k_prolong_full, dim3(grid_for((long long)nf * nf * nf, 256)), dim3(256), 0,
                     s, nc, coarse, fine);
}

__global__ void k_inject_full(int nf, const double* __restrict__ f, int nc,
                              double* __restrict__ c) {
  const long long N = (long long)nc * nc * nc;
  const int st = (nf - 1) / (nc - 1);
  for (long long i = (long long)blockIdx.x * blockDim.x + threadIdx.x; i < N;
       i += (long long)gridDim.x * blockDim.x) {
    const int jx = (int)(i / ((long long)nc * nc)), jy = (int)((i / nc) % nc), jz = (int)(i % nc);
    c[i] = f[((size_t)jx * st * nf + (size_t)jy * st) * nf + (size_t)jz * st];
  }
}
void inject_full(int nf, const double* fine, int nc, double* coarse, hipStream_t s) {
  hipLaunchKernelGGL(k_inject_full, dim3(grid_for((long long)nc * nc * nc, 256)), dim3(256), 0,
                     s, nf, fine, nc, coarse);
}

__global__ void k_add_mask(int n, const double* __restrict__ f, const double* __restrict__ u,
                           double* __restrict__ out) {
  const long long N = (long long)n * n * n;
  for (long long i = (long long)blockIdx.x * blockDim.x + threadIdx.x; i < N;
       i += (long long)gridDim.x * blockDim.x) {
    const int ix = (int)(i / ((long long)n * n)), iy = (int)((i / n) % n), iz = (int)(i % n);
    out[i] = interior(n, ix, iy, iz) ? (f ? f[i] : 0.0) + u[i] : 0.0;
  }
}
void add_mask(int n, const double* f, const double* u, double* out, hipStream_t s) {
  hipLaunchKernelGGL(k_add_mask, dim3(grid_for((long long)n * n * n, 256)), dim3(256), 0, s, n, f,
                     u, out);
}

__global__ void k_axpy_full(long long N, double a, const double* __restrict__ x,
                            double* __restrict__ y) {
  for (long long i = (long long)blockIdx.x * blockDim.x + threadIdx.x; i < N;
       i += (long long)gridDim.x * blockDim.x)
    y[i] += a * x[i];
}
void axpy_full(int n, double a, const double* x, double* y, hipStream_t s) {
  const long long N = (long long)n * n * n;
  hipLaunchKernelGGL(k_axpy_full, dim3(grid_for(N, 256)), dim3(256), 0, s, N, a, x, y);
}

__global__ void __launch_bounds__(256)
    k_dot_blocks(long long N, const double* __restrict__ a, const double* __restrict__ b,
                 double* __restrict__ part) {
  __shared__ double sred[4];
  double acc = 0.0;
  for (long long i = (long long)blockIdx.x * 256 + threadIdx.x; i < N; i += (long long)RED_BLOCKS * 256)
    acc += a[i] * b[i];
  const double s = block_sum<256>(acc, sred);
  if (threadIdx.x == 0) part[blockIdx.x] = s;
}
void dot_blocks(long long N, const double* a, const double* b, double* part, hipStream_t s) {
  hipLaunchKernelGGL(k_dot_blocks, dim3(RED_BLOCKS), dim3(256), 0, s, N, a, b, part);
}

__global__ void k_box_step(int n, double* __restrict__ u, const double* __restrict__ g, double tau,
                           double lo, double hi, int use_box) {
  const long long N = (long long)n * n * n;
  for (long long i = (long long)blockIdx.x * blockDim.x + threadIdx.x; i < N;
       i += (long long)gridDim.x * blockDim.x) {
    const int ix = (int)(i / ((long long)n * n)), iy = (int)((i / n) % n), iz = (int)(i % n);
    if (!interior(n, ix, iy, iz)) continue;
    double v = u[i] - tau * g[i];
    if (use_box) v = fmin(fmax(v, lo), hi);
    u[i] = v;
  }
}
void box_step(int n, double* u, const double* g, double tau, double lo, double hi, int use_box,
              hipStream_t s) {
  hipLaunchKernelGGL(k_box_step, dim3(grid_for((long long)n * n * n, 256)), dim3(256), 0, s, n, u,
                     g, tau, lo, hi, use_box);
}

__global__ void k_nonfinite(long long count, const double* __restrict__ x, int* flag) {
  int bad = 0;
  for (long long i = (long long)blockIdx.x * blockDim.x + threadIdx.x; i < count;
       i += (long long)gridDim.x * blockDim.x)
    if (!isfinite(x[i])) bad = 1;
  if (bad) atomicOr(flag, 1);
}
void nonfinite_flag(long long count, const double* x, int* flag, hipStream_t s) {
  if (count <= 0) return;
  hipLaunchKernelGGL(k_nonfinite, dim3(grid_for(count, 256)), dim3(256), 0, s, count, x, flag);
}

__global__ void k_copy_rows(long long total, const double* __restrict__ src,
                            double* __restrict__ dst) {
  for (long long i = (long long)blockIdx.x * blockDim.x + threadIdx.x; i < total;
       i += (long long)gridDim.x * blockDim.x)
    dst[i] = src[i];
}
void copy_elems(long long count, const double* src, double* dst, hipStream_t s) {
  if (count <= 0) return;
  hipLaunchKernelGGL(k_copy_rows, dim3(grid_for(count, 256)), dim3(256), 0, s, count, src, dst);
}
void copy_rows(int n, int rows, const double* src, double* dst, hipStream_t s) {
  copy_elems(lay_row(n) * rows, src, dst, s);
}
__global__ void k_replicate_slots(int p0, int count, int pc, const int* __restrict__ poff,
                                  double* __restrict__ partial) {
  const long long total = (long long)(count - 1) * pc;
  for (long long i = (long long)blockIdx.x * blockDim.x + threadIdx.x; i < total;
       i += (long long)gridDim.x * blockDim.x) {
    const int p = p0 + 1 + (int)(i / pc), t = (int)(i % pc);
    partial[poff[p] + t] = partial[poff[p0] + t];
  }
}
void replicate_slots(int p0, int count, int pc, const int* poff, double* partial, hipStream_t s) {
  if (count <= 1 || pc <= 0) return;
  const long long total = (long long)(count - 1) * pc;
  hipLaunchKernelGGL(k_replicate_slots, dim3(grid_for(total, 256)), dim3(256), 0, s, p0, count,
                     pc, poff, partial);
}

// ---------------------------------------------------------------------------
// Entropic epilogue (Sec. 2.2 estimator, Sec. 4.1 power sums).
// ---------------------------------------------------------------------------
// s = max Phi over every solve; w = exp(theta (Phi - s)) in FP64.
__global__ void __launch_bounds__(1024)
    k_shift_weights(int nprob, const double* __restrict__ phi, double theta,
                    double* __restrict__ w, double* s_out) {
  __shared__ double sm[1024];
  double m = -INFINITY;
  for (int p = threadIdx.x; p < nprob; p += 1024) m = fmax(m, phi[p]);
  sm[threadIdx.x] = m;
  __syncthreads();
  for (int o = 512; o > 0; o >>= 1) {
    if (threadIdx.x < o) sm[threadIdx.x] = fmax(sm[threadIdx.x], sm[threadIdx.x + o]);
    __syncthreads();
  }
  const double s = sm[0];
  for (int p = threadIdx.x; p < nprob; p += 1024) w[p] = exp(theta * (phi[p] - s));
  if (threadIdx.x == 0) *s_out = s;
}
void shift_weights(int nprob, const double* phi, double theta, double* w, double* s_out,
                   hipStream_t s) {
  hipLaunchKernelGGL(k_shift_weights, dim3(1), dim3(1024), 0, s, nprob, phi, theta, w, s_out);
}

constexpr int SB = 32;  // samples per block of the level reductions
int level_sample_blocks(int M) { return (M + SB - 1) / SB; }

// dX_m(v) = w_f[m] p_f[m](v) - w_c[m] (P p_c[m])(v) at interior v = (ix, iy, iz)
// of the fine grid; p_f and p_c are solver rows.  The addressing of a vertex
// is formed once (DxSite) and serves every sample: the fine element offset in
// a row, the coarse corner (ix/2, iy/2, iz/2) and the steps to the corners
// one further along each odd axis, with 0/1 masks, so that every sample adds
// the same corners in prolong_at's order (a masked corner adds 0).
struct DxSite {
  uint32_t of, oc, dz, dy, dx;
  double w, mz, my, mx;
};
__device__ __forceinline__ DxSite dx_site(int nf, int ix, int iy, int iz) {
  DxSite t;
  t.of = (uint32_t)(ix * nf + iy) * (uint32_t)lay_pitch(nf) + (uint32_t)(iz + lay_off(nf));
  const int nc = (nf - 1) / 2 + 1, cp = lay_pitch(nc);
  t.oc = (uint32_t)((ix >> 1) * nc + (iy >> 1)) * (uint32_t)cp + (uint32_t)((iz >> 1) + lay_off(nc));
  t.dz = iz & 1;
  t.dy = (iy & 1) ? (uint32_t)cp : 0u;
  t.dx = (ix & 1) ? (uint32_t)nc * (uint32_t)cp : 0u;
  t.mz = (iz & 1) ? 1.0 : 0.0;
  t.my = (iy & 1) ? 1.0 : 0.0;
  t.mx = (ix & 1) ? 1.0 : 0.0;
  t.w = ((ix & 1) ? 0.5 : 1.0) * ((iy & 1) ? 0.5 : 1.0) * ((iz & 1) ? 0.5 : 1.0);
  return t;
}
__device__ __forceinline__ double dx_eval(const DxSite& t, int m, size_t sf, size_t scs,
                                          const double* __restrict__ pf,
                                          const double* __restrict__ wf,
                                          const double* __restrict__ pc,
                                          const double* __restrict__ wc) {
  double d = wf[m] * pf[(size_t)m * sf + t.of];
  if (pc) {
    const double* __restrict__ c = pc + (size_t)m * scs + t.oc;
    const double c0 = c[0], c1 = c[t.dz], c2 = c[t.dy], c3 = c[t.dy + t.dz];
    const double c4 = c[t.dx], c5 = c[t.dx + t.dz], c6 = c[t.dx + t.dy],
                 c7 = c[t.dx + t.dy + t.dz];
    const double myz = t.my * t.mz, mxz = t.mx * t.mz, mxy = t.mx * t.my;
    double v = c0;
    v += t.mz * c1;
    v += t.my * c2;
    v += myz * c3;
    v += t.mx * c4;
    v += mxz * c5;
    v += mxy * c6;
    v += mxy * t.mz * c7;
    d -= wc[m] * (t.w * v);
  }
  return d;
}

// interior vertex v < nf^3 (dense index) as (ix, iy, iz); false off the interior
__device__ __forceinline__ bool dx_vertex(int nf, uint32_t v, int& ix, int& iy, int& iz) {
  const uint32_t n = (uint32_t)nf, nn = n * n;
  ix = (int)(v / nn);
  const uint32_t r = v - (uint32_t)ix * nn;
  iy = (int)(r / n);
  iz = (int)(r - (uint32_t)iy * n);
  return interior(nf, ix, iy, iz);
}

__global__ void k_level_dx_partial(int nf, int M, const double* __restrict__ pf,
                                   const double* __restrict__ wf, const double* __restrict__ pc,
                                   const double* __restrict__ wc, double* __restrict__ part) {
  const long long N = (long long)nf * nf * nf;
  const long long v = (long long)blockIdx.x * blockDim.x + threadIdx.x;
  const int sb = blockIdx.y;
  if (v >= N) return;
  int ix, iy, iz;
  double acc = 0.0;
  if (dx_vertex(nf, (uint32_t)v, ix, iy, iz)) {
    const DxSite t = dx_site(nf, ix, iy, iz);
    const size_t sf = (size_t)lay_row(nf), scs = (size_t)lay_row((nf - 1) / 2 + 1);
    const int m1 = min(M, (sb + 1) * SB);
    for (int m = sb * SB; m < m1; ++m) acc += dx_eval(t, m, sf, scs, pf, wf, pc, wc);
  }
  part[(size_t)sb * N + v] = acc;
}
void level_dx_partial(int nf, int M, const double* pf, const double* wf, const double* pc,
                      const double* wc, double* part, hipStream_t s) {
  const long long N = (long long)nf * nf * nf;
  hipLaunchKernelGGL(k_level_dx_partial, dim3(cdiv(N, 256), level_sample_blocks(M)), dim3(256),
                     0, s, nf, M, pf, wf, pc, wc, part);
}

__global__ void k_level_dx_mean(long long N, int nsb, int M, const double* __restrict__ part,
                                double* __restrict__ mean) {
  for (long long v = (long long)blockIdx.x * blockDim.x + threadIdx.x; v < N;
       v += (long long)gridDim.x * blockDim.x) {
    double acc = 0.0;
    for (int sb = 0; sb < nsb; ++sb) acc += part[(size_t)sb * N + v];
    mean[v] = acc / (double)M;
  }
}
void level_dx_mean(int nf, int M, const double* part, double* mean, hipStream_t s) {
  const long long N = (long long)nf * nf * nf;
  hipLaunchKernelGGL(k_level_dx_mean, dim3(grid_for(N, 256)), dim3(256), 0, s, N,
                     level_sample_blocks(M), M, part, mean);
}

// points per workgroup of the M2 reduction (two per thread: enough
// workgroups to fill the chip on the finest level, whose sample count is small)
constexpr int M2_CHUNK = 256 * 2;
int level_m2_chunks(int nf) {
  const long long N = (long long)nf * nf * nf;
  return cdiv(N, M2_CHUNK);
}
__global__ void __launch_bounds__(256)
    k_level_dx_m2(int nf, int M, const double* __restrict__ pf, const double* __restrict__ wf,
                  const double* __restrict__ pc, const double* __restrict__ wc,
                  const double* __restrict__ mean, double* __restrict__ part2) {
  __shared__ double sred[4];
  const long long N = (long long)nf * nf * nf;
  const int chunk = blockIdx.x, sb = blockIdx.y;
  const long long lo = (long long)chunk * M2_CHUNK, hi = min(N, lo + M2_CHUNK);
  const int m1 = min(M, (sb + 1) * SB);
  const size_t sf = (size_t)lay_row(nf), scs = (size_t)lay_row((nf - 1) / 2 + 1);
  double acc = 0.0;
  for (long long v = lo + threadIdx.x; v < hi; v += 256) {
    int ix, iy, iz;
    if (!dx_vertex(nf, (uint32_t)v, ix, iy, iz)) continue;
    const DxSite t = dx_site(nf, ix, iy, iz);
    const double mv = mean[v];
    for (int m = sb * SB; m < m1; ++m) {
      const double d = dx_eval(t, m, sf, scs, pf, wf, pc, wc) - mv;
      acc += d * d;
    }
  }
  const double sum = block_sum<256>(acc, sred);
  if (threadIdx.x == 0) part2[(size_t)sb * gridDim.x + chunk] = sum;
}
void level_dx_m2(int nf, int M, const double* pf, const double* wf, const double* pc,
                 const double* wc, const double* mean, double* part2, hipStream_t s) {
  hipLaunchKernelGGL(k_level_dx_m2, dim3(level_m2_chunks(nf), level_sample_blocks(M)), dim3(256),
                     0, s, nf, M, pf, wf, pc, wc, mean, part2);
}

// Fixed-order block sum of f(i) over i in [0, count) for 1024 threads.
template <typename F>
__device__ double block_sum_1024(int count, F f, double* sm) {
  double acc = 0.0;
  for (int i = threadIdx.x; i < count; i += 1024) acc += f(i);
  sm[threadIdx.x] = acc;
  __syncthreads();
  for (int o = 512; o > 0; o >>= 1) {
    if (threadIdx.x < o) sm[threadIdx.x] += sm[threadIdx.x + o];
    __syncthreads();
  }
  const double r = sm[0];
  __syncthreads();
  return r;
}

// Level statistics, E^ML[Y], truncation, objective (shifted units).
__global__ void __launch_bounds__(1024)
    k_epilogue_scalars(int L, const EpiLevel* __restrict__ lev, const double* __restrict__ phi,
                       const double* __restrict__ w, const double* __restrict__ part,
                       long long u_off, int nL, double theta, double alpha, int with_dx,
                       EpiOut* out) {
  __shared__ double sm[1024];
  const double s = out->s;
  double EY = 0.0, Ephi = 0.0;
  for (int i = 0; i < L; ++i) {
    const EpiLevel lv = lev[i];
    const double invM = 1.0 / (double)lv.M;
    const bool hc = lv.coarse_off >= 0;
    auto dY = [&](int m) {
      return w[lv.fine_off + m] - (hc ? w[lv.coarse_off + m] : 0.0);
    };
    const double mdy = block_sum_1024(lv.M, dY, sm) * invM;
    const double m2y = block_sum_1024(
        lv.M, [&](int m) { const double d = dY(m) - mdy; return d * d; }, sm);
    const double mphi = block_sum_1024(lv.M, [&](int m) { return phi[lv.fine_off + m]; }, sm) * invM;
    const double mdphi =
        block_sum_1024(lv.M, [&](int m) {
          return phi[lv.fine_off + m] - (hc ? phi[lv.coarse_off + m] : 0.0);
        }, sm) * invM;
    double m2x = 0.0, nmx = 0.0;
    if (with_dx) {
      const double hf = 1.0 / (double)(lv.nf - 1);
      const double h3 = hf * hf * hf;
      m2x = h3 * block_sum_1024(lv.m2_cnt, [&](int j) { return part[lv.m2_off + j]; }, sm);
      nmx = h3 * block_sum_1024(RED_BLOCKS, [&](int j) { return part[lv.nm_off + j]; }, sm);
    }
    if (threadIdx.x == 0) {
      out->mean_dY[i] = mdy;
      out->m2_dY[i] = m2y;
      out->mean_phi_f[i] = mphi;
      out->m2_dX[i] = m2x;
      out->norm2_mean_dX[i] = nmx;
    }
    EY += mdy;
    Ephi += mdphi;
  }
  const double hL = 1.0 / (double)(nL - 1);
  const double un =
      hL * hL * hL * block_sum_1024(RED_BLOCKS, [&](int j) { return part[u_off + j]; }, sm);
  if (threadIdx.x == 0) {
    const double floor_ = exp(-theta * s);
    out->EY = EY;
    out->unorm2 = un;
    out->truncated = (theta > 0.0) && (EY < floor_);
    out->denom = (theta > 0.0) ? fmax(EY, floor_) : 1.0;
    out->J = (theta > 0.0) ? s + log(out->denom) / theta + 0.5 * alpha * un
                           : Ephi + 0.5 * alpha * un;
  }
}
void epilogue_scalars(int L, const EpiLevel* lev, const double* phi, const double* w,
                      const double* part, long long u_off, int nL, double theta, double alpha,
                      int with_dx, EpiOut* out, hipStream_t s) {
  hipLaunchKernelGGL(k_epilogue_scalars, dim3(1), dim3(1024), 0, s, L, lev, phi, w, part, u_off,
                     nL, theta, alpha, with_dx, out);
}


__global__ void k_final_grad(int n, const double* __restrict__ acc, const double* __restrict__ u,
                             const EpiOut* __restrict__ eo, double alpha,
                             double* __restrict__ grad) {
  const long long N = (long long)n * n * n;
  const double inv = 1.0 / eo->denom;
  for (long long i = (long long)blockIdx.x * blockDim.x + threadIdx.x; i < N;
       i += (long long)gridDim.x * blockDim.x) {
    const int ix = (int)(i / ((long long)n * n)), iy = (int)((i / n) % n), iz = (int)(i % n);
    grad[i] = interior(n, ix, iy, iz) ? acc[i] * inv + alpha * u[i] : 0.0;
  }
}
void final_grad(int n, const double* acc, const double* u, const EpiOut* eo, double alpha,
                double* grad, hipStream_t s) {
  hipLaunchKernelGGL(k_final_grad, dim3(grid_for((long long)n * n * n, 256)), dim3(256), 0, s, n,
                     acc, u, eo, alpha, grad);
}

__global__ void k_finish_norm(int n, const double* __restrict__ part, double* dst) {
  if (threadIdx.x != 0) return;
  double acc = 0.0;
  for (int j = 0; j < RED_BLOCKS; ++j) acc += part[j];
  const double h = 1.0 / (double)(n - 1);
  *dst = h * h * h * acc;
}
void finish_norm(int n, const double* part, double* dst, hipStream_t s) {
  hipLaunchKernelGGL(k_finish_norm, dim3(1), dim3(64), 0, s, n, part, dst);
}

}  // namespace mlsgd
