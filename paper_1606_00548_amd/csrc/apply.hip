// CPR preconditioner application z = M^-1 v.
//
//   r~   = v with r~_0 = w^T v                    (quasi-IMPES decoupling)
//   dp   = V(1,1)-cycle on A_p r~_0               (pressure stage, Sec. 2.5)
//   r2   = r~ - A~(:, p) dp
//   y    = (D' + L)^-1 r2 ;  z = y - D'^-1 U z     (red-black block ILU(0))
//   z_0 += dp
//
// Variants (Sec. 2.5 names both): ABF decoupling r~ = D^-1 v per cell with
// A~ = D^-1 A, and the F-P-F composition, which first applies the block
// ILU(0) to r~ (z1), runs the two stages above on r1 = r~ - A~ z1 and adds
// z1 to the result.
//
// Kernels are templated on the preconditioner's scalar type T: double for
// the FP64 path, float for the mixed-precision path (v and z stay FP64 at
// the boundary; the coarsest pressure solve is always FP64).  Every colour
// kernel runs one thread per cell of that colour; in the colour-split
// layout all of a cell's neighbours live in the other half.
//
// V(1,1) cycle per level: red sweep from a zero guess (fused with the
// decoupling on the fine level), black sweep (which also records the black
// residuals), restriction of r - A x by 2x2x2 aggregation, coarse solve,
// black post-sweep reading the prolongated red values x + alpha e_c on the
// fly (the prolongated red values themselves are overwritten by the red
// post-sweep, so they are never stored), red post-sweep.  The smallest levels
// down to the dense coarsest solve run in one single-workgroup kernel where
// they fit its LDS (cycle_fused_level), which removes a dozen latency-bound
// launches per cycle.
#include <algorithm>

#include "internal.h"

namespace {

constexpr int FUSE_MAX = 4096;   // cells of the first level handled by the fused kernel
constexpr int DENSE_FUSED_MAX = 1024;
constexpr int DENSE_FUSED_NC = 128;   // coarsest cells of the single-workgroup kernel (cycle_fused_level)
constexpr int DENSE_PF = 17;     // coarsest-inverse entries per thread (of 1024) loaded at the fused kernel's start
constexpr int STAGE_UNROLL = 8;  // loads per thread in flight while the fused kernel stages its levels
constexpr int MAXLV = 16;
// Threads per workgroup of the per-cell kernels (sweeps, restriction,
// decoupling): one wave per workgroup streams their planes faster than four.
constexpr int SB = 64;

template <typename T>
struct Pre;
template <>
struct Pre<double> {
  static const double* R0(const cpr_ctx* c) { return c->R0; }
  static const double* J(const cpr_ctx* c) { return c->opt.decoupling == CPR_DECOUPLE_ABF ? c->Jt : c->J; }
  static double* Rt(cpr_ctx* c) { return c->Rt; }
  static double* Z1(cpr_ctx* c) { return c->Z1; }
  static const double* Dinv(const cpr_ctx* c) { return c->Dinv; }
  static const double* A(const MGLevel& l) { return l.A; }
  static double* x(MGLevel& l) { return l.x; }
  static double* r(MGLevel& l) { return l.r; }
  static double* res(MGLevel& l) { return l.res; }
  static double* Y(cpr_ctx* c) { return c->Y; }
};
template <>
struct Pre<float> {
  static const float* R0(const cpr_ctx* c) { return c->Jf; }   // unused: full FP32 blocks
  static const float* J(const cpr_ctx* c) { return c->Jf; }
  static float* Rt(cpr_ctx* c) { return c->Rtf; }
  static float* Z1(cpr_ctx* c) { return c->Z1f; }
  static const float* Dinv(const cpr_ctx* c) { return c->Dinvf; }
  static const float* A(const MGLevel& l) { return l.Af; }
  static float* x(MGLevel& l) { return l.xf; }
  static float* r(MGLevel& l) { return l.rf; }
  static float* res(MGLevel& l) { return l.resf; }
  static float* Y(cpr_ctx* c) { return c->Yf; }
};

// Decoupled block entry (d, r, c) of cell t (tiled arrays).  FP64: row 0
// lives in R0 (7 b planes), rows >= 1 in J (7 b^2 planes); FP32: the copy
// holds the full decoupled blocks (7 b^2 planes).
template <int B, typename T>
__device__ inline T at_blk(const T* __restrict__ J, const T* __restrict__ R0, size_t N, int d, int r,
                           int c, int t) {
  if constexpr (sizeof(T) == 8) {
    return r == 0 ? ldnt(R0 + tix(7 * B, d * B + c, t)) : ldnt(J + tix(7 * B * B, (d * B + r) * B + c, t));
  } else {
    return ldnt(J + tix(7 * B * B, (d * B + r) * B + c, t));
  }
}

// ------------------------------------------------------------ per-cell steps

// red cell q: x = r / a_0 (zero initial guess: every neighbour is black = 0)
template <typename T>
__device__ inline void red_zero_cell(const T* __restrict__ A, const T* __restrict__ r, T* __restrict__ x,
                                     int q) {
  x[q] = r[q] / A[q];
}

// Stencil coefficients are read non-temporally by the multi-block sweeps,
// which stream them once, and through the caches by the single-workgroup
// kernel, which reads its small levels several times.
template <bool NT, typename T>
__device__ inline T ldc(const T* p) {
  if constexpr (NT) return ldnt(p); else return *p;
}

// sum_{d>0} a_d x_nb for a colour-split cell (branch-free, missing
// neighbours masked)
template <typename T, bool NT = true>
__device__ inline T offdiag_sum(const Lay& L, const T* __restrict__ A, const T* __restrict__ x, int t) {
  CsCell cc = cs_decode(L, t);
  int nbr[7];
  bool ok[7];
  cs_nbrs(L, t, cc, nbr, ok);
  T a[7];
#pragma unroll
  for (int d = 1; d < 7; ++d) a[d] = ldc<NT>(A + (size_t)d * L.n + t);
  T s = 0;
#pragma unroll
  for (int d = 1; d < 7; ++d) {
    T v = x[nbr[d]];
    s += a[d] * (ok[d] ? v : (T)0);
  }
  return s;
}

// black cell q: Gauss-Seidel update and (RES) its residual r - A x afterwards
template <typename T, bool NT = true, bool RES = true>
__device__ inline void black_pre_cell(const Lay& L, const T* __restrict__ A, const T* __restrict__ r,
                                      T* __restrict__ x, T* __restrict__ res, int q) {
  int t = L.nh + q;
  T s = offdiag_sum<T, NT>(L, A, x, t);
  T xb = (r[t] - s) / A[t];
  x[t] = xb;
  if (RES) res[q] = r[t] - (A[t] * xb + s);
}

// black cell q after the coarse correction: neighbours are red cells whose
// corrected value is x + alpha e_c[aggregate]
template <typename T, bool NT = true>
__device__ inline void black_post_cell(const Lay& F, const Lay& C, T alpha, const T* __restrict__ A,
                                       const T* __restrict__ r, const T* __restrict__ ec,
                                       T* __restrict__ x, int q) {
  int t = F.nh + q;
  CsCell cc = cs_decode(F, t);
  int nbr[7];
  bool ok[7];
  cs_nbrs(F, t, cc, nbr, ok);
  T a[7];
#pragma unroll
  for (int d = 1; d < 7; ++d) a[d] = ldc<NT>(A + (size_t)d * F.n + t);
  T s = 0;
#pragma unroll
  for (int d = 1; d < 7; ++d) {
    int di, dj, dk;
    dir_offset(d, di, dj, dk);
    // a missing neighbour looks up the cell's own aggregate (in bounds) and is masked
    int gi = ok[d] ? cc.i + di : cc.i, gj = ok[d] ? cc.j + dj : cc.j, gk = ok[d] ? cc.k + dk : cc.k;
    T e = ec[lay_index(C, gi >> 1, gj >> 1, gk >> 1)];
    T v = x[nbr[d]] + alpha * e;
    s += a[d] * (ok[d] ? v : (T)0);
  }
  x[t] = (r[t] - s) / A[t];
}

// red cell q, general Gauss-Seidel update
template <typename T, bool NT = true>
__device__ inline void red_cell(const Lay& L, const T* __restrict__ A, const T* __restrict__ r,
                                T* __restrict__ x, int q) {
  T s = offdiag_sum<T, NT>(L, A, x, q);
  x[q] = (r[q] - s) / A[q];
}

// ------------------------------------------------------------ multi-block kernels

// Fine level entry: r~_0 = w^T v for every cell, and the zero-guess red
// sweep x_r = r~_0 / a_0.  If nrm2 is given, the input is an unnormalised
// Krylov vector: it is divided by sqrt(*nrm2) and written back first.  If
// redc is given as well, its red half is *redc times that of v0.
template <int B, typename T>
__global__ __launch_bounds__(256) void decouple_red_kernel(int n, int nh, const double* __restrict__ w,
                                                           const double* vin, double* vout,
                                                           const double* __restrict__ nrm2, const double* v0,
                                                           const double* __restrict__ redc,
                                                           const T* __restrict__ A, T* __restrict__ rp,
                                                           T* __restrict__ x) {
  int t = blockIdx.x * blockDim.x + threadIdx.x;
  if (t >= n) return;
  double hn = nrm2 ? sqrt(*nrm2) : 1.0;
  const bool red0 = redc && t < nh;
  const double rc = red0 ? *redc : 1.0;
  double s = 0.0;
#pragma unroll
  for (int r = 0; r < B; ++r) {
    double v = red0 ? rc * v0[(size_t)r * n + t] : vin[(size_t)r * n + t];
    if (nrm2) {
      v = v / hn;
      vout[(size_t)r * n + t] = v;
    }
    s = r == 0 ? v : s + w[(size_t)r * n + t] * v;   // w_0 = 1 (cpr_setup)
  }
  T rs = (T)s;
  rp[t] = rs;
  if (t < nh) x[t] = rs / A[t];
}

// The same from a natural-order vector (cpr_precond_apply), one thread per
// natural cell; rows >= 1, which stage 2 reads, are left colour-split in v.
// With the pair of stores at the end of stage 2 it saves the permuting passes
// at either end (60x220x85 oil-water, FP64: 196 -> 188 us an application).
template <int B, typename T>
__global__ __launch_bounds__(256) void decouple_nat_kernel(Lay L, const double* __restrict__ w,
                                                           const double* __restrict__ vin, double* __restrict__ v,
                                                           const T* __restrict__ A, T* __restrict__ rp,
                                                           T* __restrict__ x) {
  const int g = blockIdx.x * blockDim.x + threadIdx.x;
  if (g >= L.n) return;
  const int jk = g / L.nx, i = g - jk * L.nx;
  const int t = lay_index(L, i, jk % L.ny, jk / L.ny);
  double s = 0.0;
#pragma unroll
  for (int r = 0; r < B; ++r) {
    const double a = vin[(size_t)r * L.n + g];
    if (r > 0) v[(size_t)r * L.n + t] = a;
    s = r == 0 ? a : s + w[(size_t)r * L.n + t] * a;   // w_0 = 1 (cpr_setup)
  }
  const T rs = (T)s;
  rp[t] = rs;
  if (t < L.nh) x[t] = rs / A[t];
}

// Decoupling for ABF or for the F-P-F composition: r~ = W v per cell (ABF:
// the b x b block D_i^-1; quasi-IMPES: row 0 becomes w^T v).  Two-stage
// (P then F): r~_0 and the zero-guess red sweep as above, rows >= 1 into Rt.
// F-P-F: all of r~ into Rt, and on red cells the forward ILU step
// Z1 = D'^-1 r~ (red cells have no lower neighbours).
template <int B, typename T, bool ABF, bool FPF>
__global__ __launch_bounds__(256) void decouple_full_kernel(int n, int nh, const double* __restrict__ w,
                                                            const double* vin, double* vout,
                                                            const double* __restrict__ nrm2, const double* v0,
                                                            const double* __restrict__ redc,
                                                            const T* __restrict__ A, const T* __restrict__ Dinv,
                                                            T* __restrict__ rp, T* __restrict__ x,
                                                            T* __restrict__ Rt, T* __restrict__ Z1) {
  int t = blockIdx.x * blockDim.x + threadIdx.x;
  if (t >= n) return;
  const size_t N = n;
  double hn = nrm2 ? sqrt(*nrm2) : 1.0;
  const bool red0 = redc && t < nh;
  const double rc = red0 ? *redc : 1.0;
  double v[B], rt[B];
#pragma unroll
  for (int r = 0; r < B; ++r) {
    v[r] = red0 ? rc * v0[(size_t)r * N + t] : vin[(size_t)r * N + t];
    if (nrm2) {
      v[r] = v[r] / hn;
      vout[(size_t)r * N + t] = v[r];
    }
  }
  if constexpr (ABF) {
#pragma unroll
    for (int r = 0; r < B; ++r) {
      double s = 0.0;
#pragma unroll
      for (int c = 0; c < B; ++c) s += w[((size_t)r * B + c) * N + t] * v[c];
      rt[r] = s;
    }
  } else {
    double s = v[0];   // w_0 = 1 (cpr_setup)
#pragma unroll
    for (int r = 1; r < B; ++r) s += w[(size_t)r * N + t] * v[r];
    rt[0] = s;
#pragma unroll
    for (int r = 1; r < B; ++r) rt[r] = v[r];
  }
  if constexpr (FPF) {
    T rr[B];
#pragma unroll
    for (int r = 0; r < B; ++r) {
      rr[r] = (T)rt[r];
      Rt[(size_t)r * N + t] = rr[r];
    }
    if (t < nh) {
#pragma unroll
      for (int r = 0; r < B; ++r) {
        T a = 0;
#pragma unroll
        for (int c = 0; c < B; ++c) a += Dinv[tix(B * B, r * B + c, t)] * rr[c];
        Z1[(size_t)r * N + t] = a;
      }
    }
  } else {
    T r0 = (T)rt[0];
    rp[t] = r0;
    if (t < nh) x[t] = r0 / A[t];
#pragma unroll
    for (int r = 1; r < B; ++r) Rt[(size_t)r * N + t] = (T)rt[r];
  }
}

template <typename T, bool RES>
__global__ __launch_bounds__(256) void black_pre_kernel(Lay L, const T* __restrict__ A, const T* __restrict__ r,
                                                        T* __restrict__ x, T* __restrict__ res) {
  int q = blockIdx.x * blockDim.x + threadIdx.x;
  if (q < L.nh) black_pre_cell<T, true, RES>(L, A, r, x, res, q);
}

// Restriction: a workgroup takes 64 consecutive coarse cells in natural order
// (ci fastest) and its wave (q, s) the fine rows (2cj+q, 2ck+s) under them,
// the two fine cells (2ci, 2ci+1) of its row per lane; the four partials of a
// coarse cell meet in LDS and are combined in a fixed order.  Consecutive
// lanes so read consecutive cells of each colour half, a wave's load one run
// of 64 (with the four rows in adjacent lanes a load covered four runs of 16;
// FP64 fine level of 384x384x96: 186 -> 118 us).  Every lane takes its row's
// red cell (residual r - A x formed here) and its black cell (residual
// recorded by the black sweep) in the same order, so the lanes do not diverge
// on the colour; the two terms are added as a sum of two, whose value does not
// depend on their order.  With seq the eight residuals are summed one after the other in natural order instead, as the
// single-workgroup kernel does it (a level takes either route by its size
// and type; its values do not change with it).
// If xc is given, the coarse level's zero-guess red sweep is done here too:
// a red coarse cell stores x = r / a_0 as soon as its r is known.
template <typename T>
__global__ __launch_bounds__(256) void restrict4_kernel(Lay F, Lay C, const T* __restrict__ A,
                                                        const T* __restrict__ r, const T* __restrict__ x,
                                                        const T* __restrict__ res, T* __restrict__ rc,
                                                        const T* __restrict__ Ac, T* __restrict__ xc, int seq) {
  __shared__ T sh[4][2][64];
  const int lane = threadIdx.x & 63, sub = threadIdx.x >> 6;
  const int cn = blockIdx.x * 64 + lane;
  T lo = 0, hi = 0;   // residuals of the cells 2ci and 2ci + 1
  int ci = 0, cj = 0, ck = 0;
  if (cn < C.n) {
    const int cjk = cn / C.nx;
    ci = cn - cjk * C.nx;
    ck = cjk / C.ny;
    cj = cjk - ck * C.ny;
    const int fj = 2 * cj + (sub & 1), fk = 2 * ck + (sub >> 1);
    if (fj < F.ny && fk < F.nz) {
      const int odd = (fj + fk) & 1;
      const int fr = 2 * ci + odd, fb = 2 * ci + 1 - odd;   // red and black cell of the pair
      T vr = 0, vb = 0;
      if (fr < F.nx) {
        const int f = lay_index(F, fr, fj, fk);
        T y = A[f] * x[f] + offdiag_sum(F, A, x, f);
        vr = r[f] - y;
      }
      if (fb < F.nx) vb = res[lay_index(F, fb, fj, fk) - F.nh];
      lo = odd ? vb : vr;
      hi = odd ? vr : vb;
    }
  }
  sh[sub][0][lane] = lo;
  sh[sub][1][lane] = hi;
  __syncthreads();
  if (sub != 0 || cn >= C.n) return;
  T acc = 0;
  if (seq) {
#pragma unroll
    for (int q = 0; q < 4; ++q) {
      acc += sh[q][0][lane];
      acc += sh[q][1][lane];
    }
  } else {
    T p[4];
#pragma unroll
    for (int q = 0; q < 4; ++q) p[q] = sh[q][0][lane] + sh[q][1][lane];
    acc = (p[0] + p[2]) + (p[1] + p[3]);
  }
  const int tc = lay_index(C, ci, cj, ck);
  rc[tc] = acc;
  if (xc && tc < C.nh) red_zero_cell(Ac, rc, xc, tc);
}

template <typename T>
__global__ __launch_bounds__(256) void black_post_kernel(Lay F, Lay C, T alpha, const T* __restrict__ A,
                                                         const T* __restrict__ r, const T* __restrict__ ec,
                                                         T* __restrict__ x) {
  int q = blockIdx.x * blockDim.x + threadIdx.x;
  if (q < F.nh) black_post_cell(F, C, alpha, A, r, ec, x, q);
}

template <typename T>
__global__ __launch_bounds__(256) void red_kernel(Lay L, const T* __restrict__ A, const T* __restrict__ r,
                                                  T* __restrict__ x) {
  int q = blockIdx.x * blockDim.x + threadIdx.x;
  if (q < L.nh) red_cell(L, A, r, x, q);
}

// Coarsest level alone when the fused kernel does not take it: x = A^-1 r
// with the dense FP64 inverse (column major).  A workgroup takes GV_ROWS
// rows, so that a column's read is a whole 128-byte line, and splits the
// columns over its GV_PARTS rows of threads: the inverse (0.9 MB for 336
// cells) is read by every CU it can occupy, where one workgroup was bound by
// its own path to the L2 (5 us against about 20 of the fused kernel's 52).
constexpr int GV_ROWS = 16, GV_PARTS = 16;
template <typename T>
__global__ __launch_bounds__(GV_ROWS * GV_PARTS) void coarse_gemv_kernel(int nc, const double* __restrict__ inv,
                                                                        const T* __restrict__ r, T* __restrict__ x) {
  __shared__ double sh[GV_PARTS][GV_ROWS];
  const int lr = threadIdx.x % GV_ROWS, part = threadIdx.x / GV_ROWS;
  const int row = blockIdx.x * GV_ROWS + lr;
  double s = 0.0;
  if (row < nc) {
#pragma unroll 8
    for (int c = part; c < nc; c += GV_PARTS) s += inv[(size_t)c * nc + row] * (double)r[c];
  }
  sh[part][lr] = s;
  __syncthreads();
  if (part == 0 && row < nc) {
    double t = 0.0;
    for (int q = 0; q < GV_PARTS; ++q) t += sh[q][lr];
    x[row] = (T)t;
  }
}

// The same for a mixed solve's FP64 fallback, which keeps one order of its
// sums for good (fallback_inverse): `parts` interleaved partial sums a row (as
// many as 1,024 threads hold of nc rows), added up in turn.
template <typename T>
__global__ __launch_bounds__(1024) void coarse_parts_kernel(int nc, int parts, const double* __restrict__ inv,
                                                            const T* __restrict__ r, T* __restrict__ x) {
  __shared__ double sh[1024];
  const int rows = nc < GV_ROWS ? nc : GV_ROWS;   // a workgroup's; rows * parts <= 1,024
  const int lr = threadIdx.x % rows, part = threadIdx.x / rows;
  const int row = blockIdx.x * rows + lr;
  if (part < parts && row < nc) {
    double s = 0.0;
    for (int c = part; c < nc; c += parts) s += inv[(size_t)c * nc + row] * (double)r[c];
    sh[part * rows + lr] = s;
  }
  __syncthreads();
  if (part == 0 && row < nc) {
    double t = 0.0;
    for (int p = 0; p < parts; ++p) t += sh[p * rows + lr];
    x[row] = (T)t;
  }
}

// ------------------------------------------------------------ fused small levels

template <typename T>
struct CoarseArgs {
  int count;                 // levels handled; the last one is solved densely
  Lay lay[MAXLV];
  const T* A[MAXLV];
  T* x[MAXLV];
  T* r[MAXLV];
  // element offsets of each level's arrays in the LDS copy
  int sA[MAXLV], sx[MAXLV], sr[MAXLV], sres[MAXLV];
  const double* inv;
  T alpha;
  int pre, post;             // Gauss-Seidel sweeps before / after the coarse correction
};

// Bytes of LDS the fused kernel's copy of the levels may take (the kernel
// adds 8 KB of its own): on gfx950 a workgroup may use up to 160 KB.
constexpr int COARSE_LDS_MAX = 144 * 1024;

// The levels' stencils and the first level's right-hand side are copied into
// LDS once, every sweep, restriction and prolongation then reads and writes
// LDS, and the levels' x (and the restricted r) are copied back at the end;
// the coarsest inverse is read from global memory.  Every sweep depends on
// the one before, so with the arrays in global memory each would cost an L2
// round trip: such levels take the multi-block kernels.
template <typename T>
__global__ __launch_bounds__(1024) void coarse_cycle_kernel(CoarseArgs<T> a) {
  extern __shared__ __align__(16) unsigned char stage_raw[];
  __shared__ double part[1024];
  T* sb = reinterpret_cast<T*>(stage_raw);
  const int tid = threadIdx.x, nt = blockDim.x;
  auto Ap = [&](int l) -> const T* { return sb + a.sA[l]; };
  auto xp = [&](int l) -> T* { return sb + a.sx[l]; };
  auto rp = [&](int l) -> T* { return sb + a.sr[l]; };
  auto resp = [&](int l) -> T* { return sb + a.sres[l]; };   // residuals of the level's cells
  // The dense coarsest solve x = A^-1 r: thread (row, p) sums columns p,
  // p + parts, ... of its row, at most DENSE_PF of them.  They are loaded
  // here, so that the loads overlap the sweeps of the finer levels instead of
  // forming a chain of dependent loads at the end.
  const int nc = a.lay[a.count - 1].n;  // <= DENSE_FUSED_NC
  const int parts = nt / nc;
  const int drow = tid % nc, dp = tid / nc;
  const bool dactive = tid < nc * parts;
  double pre[DENSE_PF];
#pragma unroll
  for (int u = 0; u < DENSE_PF; ++u) {
    const int c = dp + u * parts;
    pre[u] = dactive && c < nc ? a.inv[(size_t)c * nc + drow] : 0.0;
  }
  {
    // STAGE_UNROLL independent loads per thread in flight at a time
    auto stage = [&](const T* g, T* d, int len) {
      for (int base = 0; base < len; base += STAGE_UNROLL * nt) {
        T v[STAGE_UNROLL];
#pragma unroll
        for (int u = 0; u < STAGE_UNROLL; ++u) {
          const int i = base + u * nt + tid;
          v[u] = i < len ? g[i] : (T)0;
        }
#pragma unroll
        for (int u = 0; u < STAGE_UNROLL; ++u) {
          const int i = base + u * nt + tid;
          if (i < len) d[i] = v[u];
        }
      }
    };
    for (int l = 0; l + 1 < a.count; ++l) stage(a.A[l], sb + a.sA[l], 7 * a.lay[l].n);
    stage(a.r[0], sb + a.sr[0], a.lay[0].n);
    __syncthreads();
  }
  for (int l = 0; l + 1 < a.count; ++l) {
    const Lay F = a.lay[l], C = a.lay[l + 1];
    const T* A = Ap(l);
    T *x = xp(l), *r = rp(l), *res = resp(l);
    for (int q = tid; q < F.nh; q += nt) red_zero_cell(A, r, x, q);
    __syncthreads();
    for (int q = tid; q < F.nh; q += nt) black_pre_cell<T, false>(F, A, r, x, res + F.nh, q);
    __syncthreads();
    for (int k = 1; k < a.pre; ++k) {
      for (int q = tid; q < F.nh; q += nt) red_cell<T, false>(F, A, r, x, q);
      __syncthreads();
      for (int q = tid; q < F.nh; q += nt) black_pre_cell<T, false>(F, A, r, x, res + F.nh, q);
      __syncthreads();
    }
    // restriction: the red residuals (the black sweep recorded the others),
    // one thread each, then every aggregate's sum in natural order
    T* rc = rp(l + 1);
    for (int q = tid; q < F.nh; q += nt) {
      const T y = A[q] * x[q] + offdiag_sum<T, false>(F, A, x, q);
      res[q] = r[q] - y;
    }
    __syncthreads();
    for (int tc = tid; tc < C.n; tc += nt) {
      int ci, cj, ck;
      lay_coords(C, tc, ci, cj, ck);
      T acc = 0;
      for (int fk = 2 * ck; fk <= 2 * ck + 1 && fk < F.nz; ++fk)
        for (int fj = 2 * cj; fj <= 2 * cj + 1 && fj < F.ny; ++fj)
          for (int fi = 2 * ci; fi <= 2 * ci + 1 && fi < F.nx; ++fi) acc += res[lay_index(F, fi, fj, fk)];
      rc[tc] = acc;
    }
    __syncthreads();
  }
  {
    const int L = a.count - 1;
    const T* rr = rp(L);
    if (dactive) {
      double s = 0.0;
#pragma unroll
      for (int u = 0; u < DENSE_PF; ++u) {
        const int c = dp + u * parts;
        if (c < nc) s += pre[u] * (double)rr[c];
      }
      part[tid] = s;
    }
    __syncthreads();
    T* xc = xp(L);
    for (int row = tid; row < nc; row += nt) {
      double s = 0.0;
      for (int p = 0; p < parts; ++p) s += part[p * nc + row];
      xc[row] = (T)s;
    }
    __syncthreads();
  }
  for (int l = a.count - 2; l >= 0; --l) {
    const Lay F = a.lay[l], C = a.lay[l + 1];
    const T* A = Ap(l);
    T *x = xp(l), *r = rp(l), *res = resp(l);
    const T* ec = xp(l + 1);
    for (int q = tid; q < F.nh; q += nt) black_post_cell<T, false>(F, C, a.alpha, A, r, ec, x, q);
    __syncthreads();
    for (int q = tid; q < F.nh; q += nt) red_cell<T, false>(F, A, r, x, q);
    __syncthreads();
    for (int k = 1; k < a.post; ++k) {
      for (int q = tid; q < F.nh; q += nt) black_pre_cell<T, false>(F, A, r, x, res, q);
      __syncthreads();
      for (int q = tid; q < F.nh; q += nt) red_cell<T, false>(F, A, r, x, q);
      __syncthreads();
    }
  }
  for (int l = 0; l < a.count; ++l) {
    const int n = a.lay[l].n;
    for (int i = tid; i < n; i += nt) a.x[l][i] = sb[a.sx[l] + i];
    if (l > 0)
      for (int i = tid; i < n; i += nt) a.r[l][i] = sb[a.sr[l] + i];
  }
}

// Lays out the levels' arrays in the LDS copy; returns its size in bytes.
template <typename T>
size_t coarse_stage_layout(CoarseArgs<T>& a) {
  size_t off = 0;
  for (int q = 0; q < a.count; ++q) {
    const size_t n = (size_t)a.lay[q].n;
    a.sA[q] = a.sres[q] = 0;
    if (q + 1 < a.count) {
      a.sA[q] = (int)off;
      off += 7 * n;
      a.sres[q] = (int)off;
      off += n;
    }
    a.sr[q] = (int)off;
    off += n;
    a.sx[q] = (int)off;
    off += n;
    off = (off + 1) & ~(size_t)1;   // 16-byte aligned arrays
  }
  return off * sizeof(T);
}

// The same for one smoothed level over the coarsest one (what the default
// coarsest size leaves; an aggregate has at most eight cells, so the level has
// at most PAIR_MAX), with everything but x in registers: one thread per cell,
// red ones in the first half of the workgroup, loads its stencil row,
// right-hand side and neighbours' places once, all loads in flight together,
// and a half-sweep is then six LDS reads and a division between two barriers.
// The arithmetic and its order are those above; the chains of address
// arithmetic and LDS reads of every sweep are what it saves (1,024 over 128
// cells, FP64, V(1,1): 15.8 -> 7.7 us).
constexpr int PAIR_MAX = 8 * DENSE_FUSED_NC;
template <typename T>
__global__ __launch_bounds__(1024) void coarse_pair_kernel(CoarseArgs<T> a) {
  __shared__ T xs[PAIR_MAX + 1], res[PAIR_MAX + 1], rc[DENSE_FUSED_NC], xc[DENSE_FUSED_NC + 1];
  __shared__ double part[1024];
  __shared__ unsigned short child[8 * DENSE_FUSED_NC];
  const Lay &F = a.lay[0], &C = a.lay[1];
  const int tid = threadIdx.x, nc = C.n;
  const int side = tid / (PAIR_MAX / 2), slot = tid % (PAIR_MAX / 2);   // wave-uniform side
  const bool own = slot < F.nh;
  const bool red = own && side == 0, black = own && side == 1;
  const int t = side * F.nh + (own ? slot : 0);
  T A[7];
#pragma unroll
  for (int d = 0; d < 7; ++d) A[d] = a.A[0][(size_t)d * F.n + t];
  const T r = a.r[0][t];
  const int parts = 1024 / nc, drow = tid % nc, dp = tid / nc;
  const bool dactive = tid < nc * parts;
  double pre[DENSE_PF];
#pragma unroll
  for (int u = 0; u < DENSE_PF; ++u) {
    const int c = dp + u * parts;
    pre[u] = dactive && c < nc ? a.inv[(size_t)c * nc + drow] : 0.0;
  }
  // the cell's neighbours and their aggregates as byte offsets of 16 bits, and
  // in LDS every coarse cell's aggregate; a missing cell is the zero behind
  // each array
  unsigned nbr[3], agg[3];
  {
    int nb[7], ag[7];
    bool ok[7];
    const CsCell cc = cs_decode(F, t);
    cs_nbrs(F, t, cc, nb, ok);
#pragma unroll
    for (int d = 1; d < 7; ++d) {
      int di, dj, dk;
      dir_offset(d, di, dj, dk);
      nb[d] = ok[d] ? nb[d] : PAIR_MAX;
      ag[d] = ok[d] ? lay_index(C, (cc.i + di) >> 1, (cc.j + dj) >> 1, (cc.k + dk) >> 1) : DENSE_FUSED_NC;
    }
    constexpr unsigned W = sizeof(T);
#pragma unroll
    for (int h = 0; h < 3; ++h) {
      nbr[h] = nb[2 * h + 1] * W | nb[2 * h + 2] * W << 16;
      agg[h] = ag[2 * h + 1] * W | ag[2 * h + 2] * W << 16;
    }
  }
  if (tid < 8 * nc) {
    int ci, cj, ck;
    lay_coords(C, tid >> 3, ci, cj, ck);
    const int fi = 2 * ci + (tid & 1), fj = 2 * cj + ((tid >> 1) & 1), fk = 2 * ck + ((tid >> 2) & 1);
    child[tid] = (unsigned short)(fi < F.nx && fj < F.ny && fk < F.nz ? lay_index(F, fi, fj, fk) : PAIR_MAX);
  }
  if (tid == 0) xs[PAIR_MAX] = res[PAIR_MAX] = xc[DENSE_FUSED_NC] = (T)0;
  auto at = [](const T* p, const unsigned(&n)[3], int d) {   // p at offset d of 1 .. 6
    const unsigned o = (d & 1) ? n[(d - 1) / 2] & 0xffffu : n[(d - 1) / 2] >> 16;
    return *reinterpret_cast<const T*>(reinterpret_cast<const char*>(p) + o);
  };
  auto offdiag = [&] {
    T v = 0;
#pragma unroll
    for (int d = 1; d < 7; ++d) v += A[d] * at(xs, nbr, d);
    return v;
  };
  T x = 0;
  // half-sweep of the threads of one colour; the last black one before the
  // restriction leaves its residuals
  auto sweep = [&](bool mine, bool keep) {
    if (mine) {
      const T v = offdiag();
      x = (r - v) / A[0];
      xs[t] = x;
      if (keep) res[t] = r - (A[0] * x + v);
    }
    __syncthreads();
  };
  if (red) {
    x = r / A[0];
    xs[t] = x;
  }
  __syncthreads();
  sweep(black, a.pre == 1);
  for (int k = 1; k < a.pre; ++k) {
    sweep(red, false);
    sweep(black, k + 1 == a.pre);
  }
  if (red) {
    const T y = A[0] * x + offdiag();
    res[t] = r - y;
  }
  __syncthreads();
  if (tid < nc) {
    T acc = 0;
#pragma unroll
    for (int e = 0; e < 8; ++e) acc += res[child[8 * tid + e]];
    rc[tid] = acc;
    a.r[1][tid] = acc;
  }
  __syncthreads();
  if (dactive) {
    double v = 0.0;
#pragma unroll
    for (int u = 0; u < DENSE_PF; ++u) {
      const int c = dp + u * parts;
      if (c < nc) v += pre[u] * (double)rc[c];
    }
    part[tid] = v;
  }
  __syncthreads();
  if (tid < nc) {
    double v = 0.0;
    for (int p = 0; p < parts; ++p) v += part[p * nc + tid];
    xc[tid] = (T)v;
    a.x[1][tid] = (T)v;
  }
  __syncthreads();
  if (black) {
    T v = 0;
#pragma unroll
    for (int d = 1; d < 7; ++d) {
      const T p = at(xs, nbr, d) + a.alpha * at(xc, agg, d);
      v += A[d] * p;
    }
    x = (r - v) / A[0];
    xs[t] = x;
  }
  __syncthreads();
  sweep(red, false);
  for (int k = 1; k < a.post; ++k) {
    sweep(black, false);
    sweep(red, false);
  }
  if (own) a.x[0][t] = x;
}

template <typename T>
bool coarse_pair(const CoarseArgs<T>& a) {
  return a.count == 2 && a.lay[1].n <= DENSE_FUSED_NC && a.lay[0].n <= PAIR_MAX;
}

template <typename T>
hipError_t launch_coarse_cycle(CoarseArgs<T>& a, hipStream_t s) {
  if (coarse_pair(a)) {
    coarse_pair_kernel<T><<<1, 1024, 0, s>>>(a);
    return hipSuccess;
  }
  // more than the default 64 KB of dynamic LDS
  static const hipError_t big_lds = hipFuncSetAttribute(
      (const void*)coarse_cycle_kernel<T>, hipFuncAttributeMaxDynamicSharedMemorySize, COARSE_LDS_MAX);
  if (big_lds != hipSuccess) return big_lds;
  coarse_cycle_kernel<T><<<1, 1024, coarse_stage_layout(a), s>>>(a);
  return hipSuccess;
}

// ------------------------------------------------------------ stage 2 + block ILU(0)

template <int B, typename T>
__device__ inline void offdiag_apply(const Lay& L, int t, const CsCell& cc, const T* J, const T* R0,
                                     const T* __restrict__ Y, T (&s)[B]) {
  const size_t N = L.n;
  int nbr[7];
  bool ok[7];
  cs_nbrs(L, t, cc, nbr, ok);
  T a[7][B][B];
#pragma unroll
  for (int d = 1; d < 7; ++d)
#pragma unroll
    for (int r = 0; r < B; ++r)
#pragma unroll
      for (int c = 0; c < B; ++c) a[d][r][c] = at_blk<B, T>(J, R0, N, d, r, c, t);
#pragma unroll
  for (int r = 0; r < B; ++r) s[r] = 0;
#pragma unroll
  for (int d = 1; d < 7; ++d) {
    T y[B];
#pragma unroll
    for (int c = 0; c < B; ++c) {
      T v = Y[c * N + nbr[d]];
      y[c] = ok[d] ? v : (T)0;
    }
#pragma unroll
    for (int r = 0; r < B; ++r) {
      T acc = 0;
#pragma unroll
      for (int c = 0; c < B; ++c) acc += a[d][r][c] * y[c];
      s[r] += acc;
    }
  }
}

template <int B, typename T>
__device__ inline void dinv_apply(const T* __restrict__ Dinv, size_t N, int t, const T (&in)[B], T (&out)[B]) {
#pragma unroll
  for (int r = 0; r < B; ++r) {
    T a = 0;
#pragma unroll
    for (int c = 0; c < B; ++c) a += Dinv[tix(B * B, r * B + c, t)] * in[c];
    out[r] = a;
  }
}

// Stage 2 reads rows >= 1 of the decoupled residual from v: the Krylov
// vector itself for quasi-IMPES P-then-F (VT = double), the decoupled
// residual Rt otherwise (VT = T).  With z1 given (F-P-F) the first stage's
// result is added to z.

// red cells: forward ILU step y_r = D'^-1 r2_r (no lower neighbours).  With
// SWEEP the last Gauss-Seidel half-sweep of the pressure cycle comes first:
// dp = (r~_0 - sum_d a_d dp_nb) / a_0 with the stencil a_d = A~_d(0, 0), the
// values stage 2 needs itself, so the sweep's own pass (its stencil planes,
// right-hand side and neighbours: 10 of 50 values a cell in FP64) and launch
// are saved (FP64, 384x384x96: 98 + 388 us apart, 391 us together).
template <int B, typename T, typename VT, bool SWEEP>
__global__ __launch_bounds__(256) void stage2_red_fwd_kernel(Lay L, const T* __restrict__ J,
                                                             const T* __restrict__ R0,
                                                             const T* __restrict__ Dinv,
                                                             const VT* __restrict__ v,
                                                             const T* __restrict__ rp, T* dp, T* __restrict__ Y) {
  int t = blockIdx.x * blockDim.x + threadIdx.x;
  if (t >= L.nh) return;
  CsCell cc = cs_decode(L, t);
  const size_t N = L.n;
  int nbr[7];
  bool ok[7];
  cs_nbrs(L, t, cc, nbr, ok);
  T a[7][B];
#pragma unroll
  for (int d = 0; d < 7; ++d)
#pragma unroll
    for (int r = 0; r < B; ++r) a[d][r] = at_blk<B, T>(J, R0, N, d, r, 0, t);
  T r2[B], y[B], p[7];
  r2[0] = rp[t];
#pragma unroll
  for (int r = 1; r < B; ++r) r2[r] = (T)v[r * N + t];
#pragma unroll
  for (int d = SWEEP ? 1 : 0; d < 7; ++d) {
    const T q = dp[nbr[d]];
    p[d] = ok[d] ? q : (T)0;
  }
  if (SWEEP) {
    T s = 0;
#pragma unroll
    for (int d = 1; d < 7; ++d) s += a[d][0] * p[d];
    p[0] = (r2[0] - s) / a[0][0];
    dp[t] = p[0];
  }
#pragma unroll
  for (int d = 0; d < 7; ++d)
#pragma unroll
    for (int r = 0; r < B; ++r) r2[r] -= a[d][r] * p[d];
  dinv_apply<B, T>(Dinv, L.n, t, r2, y);
#pragma unroll
  for (int r = 0; r < B; ++r) Y[(size_t)r * L.n + t] = y[r];
}

// black cells: y_b = D'^-1 (r2_b - sum_red A~_bk y_k); no upper neighbours,
// so z_b = y_b (+ dp on the pressure unknown)
template <int B, typename T, typename VT>
__global__ __launch_bounds__(256) void stage2_black_kernel(Lay L, const T* __restrict__ J,
                                                           const T* __restrict__ R0,
                                                           const T* __restrict__ Dinv,
                                                           const VT* __restrict__ v,
                                                           const T* __restrict__ rp,
                                                           const T* __restrict__ dp, T* __restrict__ Y,
                                                           const T* __restrict__ z1,
                                                           double* __restrict__ z) {
  int q = blockIdx.x * blockDim.x + threadIdx.x;
  if (q >= L.nh) return;
  int t = L.nh + q;
  CsCell cc = cs_decode(L, t);
  const size_t N = L.n;
  // r2 = r~ - A~(:,p) dp and s = sum_red A~_bk y_k, each off-diagonal block
  // read once (branch-free, non-temporal; missing neighbours masked)
  int nbr[7];
  bool ok[7];
  cs_nbrs(L, t, cc, nbr, ok);
  T a[7][B][B];
#pragma unroll
  for (int d = 0; d < 7; ++d)
#pragma unroll
    for (int r = 0; r < B; ++r)
#pragma unroll
      for (int c = 0; c < B; ++c)
        a[d][r][c] = (d == 0 && c > 0) ? (T)0 : at_blk<B, T>(J, R0, N, d, r, c, t);
  T r2[B], s[B], y[B];
  r2[0] = rp[t];
#pragma unroll
  for (int r = 1; r < B; ++r) r2[r] = (T)v[r * N + t];
  {
    T p = dp[t];
#pragma unroll
    for (int r = 0; r < B; ++r) r2[r] -= a[0][r][0] * p;
  }
#pragma unroll
  for (int r = 0; r < B; ++r) s[r] = 0;
#pragma unroll
  for (int d = 1; d < 7; ++d) {
    T p = dp[nbr[d]];
    p = ok[d] ? p : (T)0;
    T yk[B];
#pragma unroll
    for (int c = 0; c < B; ++c) {
      T vv = Y[c * N + nbr[d]];
      yk[c] = ok[d] ? vv : (T)0;
    }
#pragma unroll
    for (int r = 0; r < B; ++r) {
      r2[r] -= a[d][r][0] * p;
      T acc = a[d][r][0] * yk[0];
#pragma unroll
      for (int c = 1; c < B; ++c) acc += a[d][r][c] * yk[c];
      s[r] += acc;
    }
  }
#pragma unroll
  for (int r = 0; r < B; ++r) r2[r] -= s[r];
  dinv_apply<B, T>(Dinv, L.n, t, r2, y);
#pragma unroll
  for (int r = 0; r < B; ++r) Y[r * N + t] = y[r];
  z[t] = (double)y[0] + (double)dp[t];
#pragma unroll
  for (int r = 1; r < B; ++r) z[r * N + t] = (double)y[r];
  if (z1) {
#pragma unroll
    for (int r = 0; r < B; ++r) z[r * N + t] += (double)z1[r * N + t];
  }
}

// red cells, backward step: z_r = y_r - D'^-1 sum_black A~_rk y_k.  NAT: z is
// stored in natural order in zn, with the black cell's of the same pair along
// x, one of the cell's neighbours.
template <int B, typename T, bool NAT>
__global__ __launch_bounds__(256) void stage2_red_bwd_kernel(Lay L, const T* __restrict__ J,
                                                             const T* __restrict__ R0,
                                                             const T* __restrict__ Dinv,
                                                             const T* __restrict__ dp,
                                                             const T* __restrict__ Y,
                                                             const T* __restrict__ z1,
                                                             double* __restrict__ z, double* __restrict__ zn) {
  int t = blockIdx.x * blockDim.x + threadIdx.x;
  if (t >= L.nh) return;
  CsCell cc = cs_decode(L, t);
  T s[B], u[B];
  offdiag_apply<B, T>(L, t, cc, J, R0, Y, s);
  dinv_apply<B, T>(Dinv, L.n, t, s, u);
  const size_t N = L.n;
  if (NAT) {
    const size_t row = (size_t)L.nx * (cc.j + (size_t)L.ny * cc.k);
#pragma unroll
    for (int r = 0; r < B; ++r) {
      const double zr = r == 0 ? (double)(Y[t] - u[0]) + (double)dp[t] : (double)(Y[r * N + t] - u[r]);
      const double zb = z[r * N + L.nh + t];
      zn[r * N + row + cc.i] = zr;
      zn[r * N + row + (cc.i ^ 1)] = zb;
    }
    return;
  }
  z[t] = (double)(Y[t] - u[0]) + (double)dp[t];
#pragma unroll
  for (int r = 1; r < B; ++r) z[r * N + t] = (double)(Y[r * N + t] - u[r]);
  if (z1) {
#pragma unroll
    for (int r = 0; r < B; ++r) z[r * N + t] += (double)z1[r * N + t];
  }
}

// ------------------------------------------------------------ stage 2, tiled ILU order
// The same stage with the block ILU(0) in the tiled red-black order (one
// thread per tile of 1 x 2 x 2 cells, see tile_of_thread): forward over the
// red tiles, forward and backward over the black tiles (whose neighbours in
// other tiles are all red, so their backward step only involves
// tile-mates), backward over the red tiles.  Inside a thread the tile's
// cells are taken in order q = 0..3 forward and 3..0 backward, and each
// sum over neighbours runs in direction order.

template <int B, typename T>
__device__ inline void blk_add(const T* J, const T* R0, size_t N, int d, int t, const T (&v)[B], T (&acc)[B]) {
#pragma unroll
  for (int r = 0; r < B; ++r) {
    T a = 0;
#pragma unroll
    for (int c = 0; c < B; ++c) a += at_blk<B, T>(J, R0, N, d, r, c, t) * v[c];
    acc[r] += a;
  }
}

// Forward step's right-hand side of cell t: the stage-2 residual r2 = r~ -
// A~(:, p) dp minus the sum over the earlier neighbours (early[d]) of
// A~_tk y_k (yn[d]), each block read once: the full block where the
// neighbour is earlier, its pressure column otherwise.  The residual terms
// run in direction order, and the neighbour sum is subtracted at the end.
template <int B, typename T, typename VT>
__device__ inline void stage2_fwd_rhs(const Lay& L, int t, const T* J, const T* R0, const VT* __restrict__ v,
                                      const T* __restrict__ rp, const T* __restrict__ dp, const bool (&early)[7],
                                      const T (&yn)[7][B], T (&out)[B]) {
  const size_t N = L.n;
  CsCell cc = cs_decode(L, t);
  int nbr[7];
  bool ok[7];
  cs_nbrs(L, t, cc, nbr, ok);
  T r2[B], s[B];
  r2[0] = rp[t];
#pragma unroll
  for (int r = 1; r < B; ++r) r2[r] = (T)v[r * N + t];
  {
    const T p0 = dp[t];
#pragma unroll
    for (int r = 0; r < B; ++r) r2[r] -= at_blk<B, T>(J, R0, N, 0, r, 0, t) * p0;
  }
#pragma unroll
  for (int r = 0; r < B; ++r) s[r] = 0;
#pragma unroll
  for (int d = 1; d < 7; ++d) {
    T p = dp[nbr[d]];
    p = ok[d] ? p : (T)0;
    if (early[d]) {
      T a[B][B];
#pragma unroll
      for (int r = 0; r < B; ++r)
#pragma unroll
        for (int c = 0; c < B; ++c) a[r][c] = at_blk<B, T>(J, R0, N, d, r, c, t);
#pragma unroll
      for (int r = 0; r < B; ++r) {
        r2[r] -= a[r][0] * p;
        T acc = a[r][0] * yn[d][0];
#pragma unroll
        for (int c = 1; c < B; ++c) acc += a[r][c] * yn[d][c];
        s[r] += acc;
      }
    } else {
#pragma unroll
      for (int r = 0; r < B; ++r) r2[r] -= at_blk<B, T>(J, R0, N, d, r, 0, t) * p;
    }
  }
#pragma unroll
  for (int r = 0; r < B; ++r) out[r] = r2[r] - s[r];
}

template <int B, typename T, typename VT>
__global__ __launch_bounds__(256) void stage2_tiles_red_fwd_kernel(Lay L, const T* __restrict__ J,
                                                                   const T* __restrict__ R0,
                                                                   const T* __restrict__ Dinv,
                                                                   const VT* __restrict__ v,
                                                                   const T* __restrict__ rp,
                                                                   const T* __restrict__ dp, T* __restrict__ Y) {
  int i, tj, tk;
  if (!tile_of_thread(L, 0, (long)blockIdx.x * blockDim.x + threadIdx.x, i, tj, tk)) return;
  const size_t N = L.n;
  T y[4][B];
#pragma unroll
  for (int q = 0; q < 4; ++q) {
    const int j = 2 * tj + (q & 1), k = 2 * tk + (q >> 1);
    if (j >= L.ny || k >= L.nz) continue;
    const int t = lay_index(L, i, j, k);
    // earlier neighbours of a red tile's cell: its tile-mates below q (-y, -z)
    bool early[7] = {false, false, false, (q & 1) != 0, false, (q & 2) != 0, false};
    T yn[7][B];
#pragma unroll
    for (int c = 0; c < B; ++c) {
      yn[3][c] = (q & 1) ? y[(q & 1) ? q - 1 : 0][c] : (T)0;
      yn[5][c] = (q & 2) ? y[(q & 2) ? q - 2 : 0][c] : (T)0;
    }
    T r2[B];
    stage2_fwd_rhs<B, T, VT>(L, t, J, R0, v, rp, dp, early, yn, r2);
    dinv_apply<B, T>(Dinv, N, t, r2, y[q]);
#pragma unroll
    for (int r = 0; r < B; ++r) Y[(size_t)r * N + t] = y[q][r];
  }
}

template <int B, typename T, typename VT>
__global__ __launch_bounds__(256) void stage2_tiles_black_kernel(Lay L, const T* __restrict__ J,
                                                                 const T* __restrict__ R0,
                                                                 const T* __restrict__ Dinv,
                                                                 const VT* __restrict__ v,
                                                                 const T* __restrict__ rp,
                                                                 const T* __restrict__ dp, T* __restrict__ Y,
                                                                 double* __restrict__ z) {
  int i, tj, tk;
  if (!tile_of_thread(L, 1, (long)blockIdx.x * blockDim.x + threadIdx.x, i, tj, tk)) return;
  const size_t N = L.n;
  T y[4][B];
  int tq[4];
#pragma unroll
  for (int q = 0; q < 4; ++q) {
    const int j = 2 * tj + (q & 1), k = 2 * tk + (q >> 1);
    tq[q] = (j < L.ny && k < L.nz) ? lay_index(L, i, j, k) : -1;
    if (tq[q] < 0) continue;
    const int t = tq[q];
    CsCell cc = cs_decode(L, t);
    int nbr[7];
    bool ok[7];
    cs_nbrs(L, t, cc, nbr, ok);
    // earlier neighbours: tile-mates below q, and every neighbour in another
    // tile (red); the latter's y come from the red forward kernel
    bool early[7];
    T yn[7][B];
    early[0] = false;
#pragma unroll
    for (int d = 1; d < 7; ++d) {
      const int mate = tile_mate(q, d);
      early[d] = ok[d] && mate < q;
#pragma unroll
      for (int c = 0; c < B; ++c)
        yn[d][c] = !early[d] ? (T)0 : mate >= 0 ? y[mate < 0 ? 0 : mate][c] : Y[(size_t)c * N + nbr[d]];
    }
    T r2[B];
    stage2_fwd_rhs<B, T, VT>(L, t, J, R0, v, rp, dp, early, yn, r2);
    dinv_apply<B, T>(Dinv, N, t, r2, y[q]);
  }
  // backward: only tile-mates above q are later
  T zt[4][B];
#pragma unroll
  for (int q = 3; q >= 0; --q) {
    if (tq[q] < 0) continue;
    const int t = tq[q];
    T u[B], w[B];
#pragma unroll
    for (int r = 0; r < B; ++r) u[r] = 0;
    if (!(q & 1) && tq[q + 1 > 3 ? 3 : q + 1] >= 0) blk_add<B, T>(J, R0, N, 4, t, zt[q + 1 > 3 ? 3 : q + 1], u);
    if (!(q & 2) && tq[q + 2 > 3 ? 3 : q + 2] >= 0) blk_add<B, T>(J, R0, N, 6, t, zt[q + 2 > 3 ? 3 : q + 2], u);
    dinv_apply<B, T>(Dinv, N, t, u, w);
#pragma unroll
    for (int r = 0; r < B; ++r) zt[q][r] = y[q][r] - w[r];
#pragma unroll
    for (int r = 0; r < B; ++r) Y[(size_t)r * N + t] = zt[q][r];
    z[t] = (double)zt[q][0] + (double)dp[t];
#pragma unroll
    for (int r = 1; r < B; ++r) z[(size_t)r * N + t] = (double)zt[q][r];
  }
}

template <int B, typename T>
__global__ __launch_bounds__(256) void stage2_tiles_red_bwd_kernel(Lay L, const T* __restrict__ J,
                                                                   const T* __restrict__ R0,
                                                                   const T* __restrict__ Dinv,
                                                                   const T* __restrict__ dp,
                                                                   const T* __restrict__ Y,
                                                                   double* __restrict__ z) {
  int i, tj, tk;
  if (!tile_of_thread(L, 0, (long)blockIdx.x * blockDim.x + threadIdx.x, i, tj, tk)) return;
  const size_t N = L.n;
  int tq[4];
#pragma unroll
  for (int q = 0; q < 4; ++q) {
    const int j = 2 * tj + (q & 1), k = 2 * tk + (q >> 1);
    tq[q] = (j < L.ny && k < L.nz) ? lay_index(L, i, j, k) : -1;
  }
  // later neighbours of a red tile's cell: tile-mates above q, and every
  // neighbour in another tile (black, whose z the black kernel left in Y)
  T zt[4][B];
#pragma unroll
  for (int q = 3; q >= 0; --q) {
    if (tq[q] < 0) continue;
    const int t = tq[q];
    CsCell cc = cs_decode(L, t);
    int nbr[7];
    bool ok[7];
    cs_nbrs(L, t, cc, nbr, ok);
    T u[B], w[B];
#pragma unroll
    for (int r = 0; r < B; ++r) u[r] = 0;
#pragma unroll
    for (int d = 1; d < 7; ++d) {
      if (!ok[d]) continue;
      const int mate = tile_mate(q, d);
      if (mate >= 0 && mate < q) continue;
      T zk[B];
#pragma unroll
      for (int c = 0; c < B; ++c) zk[c] = mate >= 0 ? zt[mate < 0 ? 0 : mate][c] : Y[(size_t)c * N + nbr[d]];
      blk_add<B, T>(J, R0, N, d, t, zk, u);
    }
    dinv_apply<B, T>(Dinv, N, t, u, w);
#pragma unroll
    for (int r = 0; r < B; ++r) zt[q][r] = Y[(size_t)r * N + t] - w[r];
    z[t] = (double)zt[q][0] + (double)dp[t];
#pragma unroll
    for (int r = 1; r < B; ++r) z[(size_t)r * N + t] = (double)zt[q][r];
  }
}

// ------------------------------------------------------------ F-P-F first stage
// z1 = ILU(0)^-1 r~ and the residual r1 = r~ - A~ z1 that the P-then-F
// stages then see.  ILU(0) on the 7-point graph differs from A~ only between
// black cells two steps apart (through a red cell), so r1 vanishes on red
// cells: the red backward kernel stores those zeros (and the matching zero
// initial red sweep of the V-cycle), the residual kernel runs on black cells.

// black cells: z1_b = y_b = D'^-1 (r~_b - sum_red A~_bk y_k)
template <int B, typename T>
__global__ __launch_bounds__(256) void fpf_black_kernel(Lay L, const T* __restrict__ J, const T* __restrict__ R0,
                                                        const T* __restrict__ Dinv, const T* __restrict__ Rt,
                                                        T* __restrict__ Z1) {
  int q = blockIdx.x * blockDim.x + threadIdx.x;
  if (q >= L.nh) return;
  int t = L.nh + q;
  CsCell cc = cs_decode(L, t);
  const size_t N = L.n;
  T s[B], r[B], y[B];
  offdiag_apply<B, T>(L, t, cc, J, R0, Z1, s);
#pragma unroll
  for (int e = 0; e < B; ++e) r[e] = Rt[e * N + t] - s[e];
  dinv_apply<B, T>(Dinv, L.n, t, r, y);
#pragma unroll
  for (int e = 0; e < B; ++e) Z1[e * N + t] = y[e];
}

// red cells: z1_r = y_r - D'^-1 sum_black A~_rk z1_k; r1_r = 0 (rows of Rt,
// the pressure right-hand side and the zero-guess red sweep of level 0)
template <int B, typename T>
__global__ __launch_bounds__(256) void fpf_red_bwd_kernel(Lay L, const T* __restrict__ J, const T* __restrict__ R0,
                                                          const T* __restrict__ Dinv, T* __restrict__ Z1,
                                                          T* __restrict__ Rt, T* __restrict__ rp,
                                                          T* __restrict__ x) {
  int t = blockIdx.x * blockDim.x + threadIdx.x;
  if (t >= L.nh) return;
  CsCell cc = cs_decode(L, t);
  const size_t N = L.n;
  T s[B], u[B];
  offdiag_apply<B, T>(L, t, cc, J, R0, Z1, s);
  dinv_apply<B, T>(Dinv, L.n, t, s, u);
#pragma unroll
  for (int e = 0; e < B; ++e) {
    Z1[e * N + t] = Z1[e * N + t] - u[e];
    Rt[e * N + t] = (T)0;
  }
  rp[t] = (T)0;
  x[t] = (T)0;
}

// black cells: r1_b = r~_b - A~_bb z1_b - sum_red A~_bk z1_k; row 0 is the
// pressure right-hand side, rows >= 1 overwrite Rt
template <int B, typename T>
__global__ __launch_bounds__(256) void fpf_resid_kernel(Lay L, const T* __restrict__ J, const T* __restrict__ R0,
                                                        const T* __restrict__ Z1, T* __restrict__ Rt,
                                                        T* __restrict__ rp) {
  int q = blockIdx.x * blockDim.x + threadIdx.x;
  if (q >= L.nh) return;
  int t = L.nh + q;
  CsCell cc = cs_decode(L, t);
  const size_t N = L.n;
  T s[B], r[B];
  offdiag_apply<B, T>(L, t, cc, J, R0, Z1, s);
#pragma unroll
  for (int e = 0; e < B; ++e) {
    T a = s[e];
#pragma unroll
    for (int c = 0; c < B; ++c) a += at_blk<B, T>(J, R0, N, 0, e, c, t) * Z1[c * N + t];
    r[e] = Rt[e * N + t] - a;
  }
  rp[t] = r[0];
#pragma unroll
  for (int e = 1; e < B; ++e) Rt[e * N + t] = r[e];
}

// ------------------------------------------------------------ host side

#define TIMED(cls, launch) \
  do {                     \
    prof_begin(ctx, cls);  \
    launch;                \
    prof_end(ctx, cls);    \
  } while (0)

// First of the levels small enough for a single workgroup (nl: none).  The
// learned stage runs above them (options.nn_level).
int fused_level(const cpr_ctx* ctx) {
  const int nl = (int)ctx->levels.size();
  const int nc = ctx->levels.back().lay.n;
  int fuse = nl;
  if (nc <= DENSE_FUSED_MAX && nl <= MAXLV) {
    fuse = nl - 1;
    for (int l = 1; l < nl; ++l)
      if (ctx->levels[l].lay.n <= FUSE_MAX) { fuse = l; break; }
    if (nl == 1) fuse = 0;
  }
  return fuse;
}

const double* coarsest_inverse(const cpr_ctx* ctx) {
  return mixed_fallback(ctx) && ctx->cinv64 ? ctx->cinv64 : ctx->cinv;
}

template <typename T>
CoarseArgs<T> coarse_args(cpr_ctx* ctx, int first) {
  CoarseArgs<T> a;
  a.count = (int)ctx->levels.size() - first;
  for (int q = 0; q < a.count; ++q) {
    MGLevel& L = ctx->levels[first + q];
    a.lay[q] = L.lay;
    a.A[q] = Pre<T>::A(L);
    a.x[q] = Pre<T>::x(L);
    a.r[q] = Pre<T>::r(L);
  }
  a.inv = coarsest_inverse(ctx);
  a.alpha = (T)ctx->opt.mg_alpha;
  a.pre = ctx->opt.mg_pre;
  a.post = ctx->opt.mg_post;
  return a;
}

// First level the cycle hands to the single-workgroup kernel (nl: none, and
// the coarsest solve is a kernel of its own).  The kernel saves the launches
// of its levels, but is one workgroup: it takes levels that it can hold (one
// level in registers, more in LDS up to about 1,790 cells in FP64 and 3,570 in
// FP32) over a coarsest inverse of at most DENSE_FUSED_NC rows, which its
// threads can hold in registers from the start; reading a larger one costs it
// more than the launches.  One application, V(1,1) FP64, one workgroup
// against multi-block kernels: 64 (by now 56) against 72 us with 1,024 over
// 128 cells (64x64x16), 78 against 73 with 1,600 over 200 (80x80x16), and with
// the levels in global memory 343 against 290 with 2,464 over 336 (60x220x85),
// 156 against 92 with 3,456 over 432 (96x96x24).
template <typename T>
int cycle_fused_level(cpr_ctx* ctx) {
  const int nl = (int)ctx->levels.size();
  if (ctx->levels.back().lay.n > DENSE_FUSED_NC) return nl;
  for (int l = fused_level(ctx); l + 1 < nl; ++l) {
    CoarseArgs<T> a = coarse_args<T>(ctx, l);
    if (coarse_pair(a) || coarse_stage_layout(a) <= (size_t)COARSE_LDS_MAX) return l;
  }
  return nl;
}

// The last red sweep of the fine level, left to the first kernel of stage 2:
// both run over the red cells, the sweep's stencil is the pressure column of
// the decoupled row 0 that stage 2 reads anyway, and the swept value is only
// read by this cell's own row (red cells couple to black ones).  Not where
// the fine level is solved directly or something (the learned stage) reads
// the finished cycle in between, nor with tiles as colours.
bool red_sweep_in_stage2(const cpr_ctx* ctx) {
  return ctx->levels.size() > 1 && ctx->opt.ilu_order == CPR_ILU_RED_BLACK &&
         !(learned_on(ctx) && ctx->opt.nn_level == 0);
}

template <typename T>
void vcycle(cpr_ctx* ctx, bool skip_last_red) {
  hipStream_t s = ctx->stream;
  const int nl = (int)ctx->levels.size();
  const int nc = ctx->levels.back().lay.n;
  const int small = fused_level(ctx), fuse = cycle_fused_level<T>(ctx);
  const T alpha = (T)ctx->opt.mg_alpha;
  const int down = fuse < nl ? fuse : nl - 1;   // levels smoothed by multi-block kernels
  for (int l = 0; l < down; ++l) {
    MGLevel& L = ctx->levels[l];
    MGLevel& C = ctx->levels[l + 1];
    int nh = div_up(L.lay.nh, SB);
    // level 0's zero-guess red sweep is fused into the decoupling kernel and
    // that of the coarser multi-block levels into the restriction above them;
    // the last black sweep leaves its residuals for the restriction
    auto black = [&](bool last) {
      if (last)
        TIMED(CPR_KCLASS_SMOOTH, (black_pre_kernel<T, true><<<nh, SB, 0, s>>>(L.lay, Pre<T>::A(L), Pre<T>::r(L),
                                                                              Pre<T>::x(L), Pre<T>::res(L))));
      else
        TIMED(CPR_KCLASS_SMOOTH, (black_pre_kernel<T, false><<<nh, SB, 0, s>>>(L.lay, Pre<T>::A(L), Pre<T>::r(L),
                                                                               Pre<T>::x(L), Pre<T>::res(L))));
    };
    black(ctx->opt.mg_pre == 1);
    for (int k = 1; k < ctx->opt.mg_pre; ++k) {
      TIMED(CPR_KCLASS_SMOOTH, (red_kernel<T><<<nh, SB, 0, s>>>(L.lay, Pre<T>::A(L), Pre<T>::r(L), Pre<T>::x(L))));
      black(k + 1 == ctx->opt.mg_pre);
    }
    const bool next_multi = l + 1 < down;
    restrict4_kernel<T><<<div_up(C.lay.n, 64), 256, 0, s>>>(
        L.lay, C.lay, Pre<T>::A(L), Pre<T>::r(L), Pre<T>::x(L), Pre<T>::res(L), Pre<T>::r(C),
        next_multi ? Pre<T>::A(C) : nullptr, next_multi ? Pre<T>::x(C) : nullptr, l >= small);
  }
  if (fuse < nl) {
    CoarseArgs<T> a = coarse_args<T>(ctx, fuse);
    const hipError_t e = launch_coarse_cycle<T>(a, s);
    if (e != hipSuccess) set_hip_err(ctx, e, "coarse_cycle_kernel");
  } else {
    MGLevel& L = ctx->levels.back();
    if (mixed_fallback(ctx))
      coarse_parts_kernel<T><<<div_up(nc, std::min(nc, GV_ROWS)), 1024, 0, s>>>(
          nc, nc <= DENSE_FUSED_MAX && nl <= MAXLV ? 1024 / nc : 1, coarsest_inverse(ctx), Pre<T>::r(L), Pre<T>::x(L));
    else
      coarse_gemv_kernel<T><<<div_up(nc, GV_ROWS), GV_ROWS * GV_PARTS, 0, s>>>(nc, ctx->cinv, Pre<T>::r(L),
                                                                               Pre<T>::x(L));
  }
  for (int l = down - 1; l >= 0; --l) {
    MGLevel& L = ctx->levels[l];
    MGLevel& C = ctx->levels[l + 1];
    int nh = div_up(L.lay.nh, SB);
    TIMED(CPR_KCLASS_SMOOTH, (black_post_kernel<T><<<nh, SB, 0, s>>>(L.lay, C.lay, alpha, Pre<T>::A(L),
                                                                      Pre<T>::r(L), Pre<T>::x(C), Pre<T>::x(L))));
    for (int k = 1; k <= ctx->opt.mg_post; ++k) {
      if (k > 1)
        TIMED(CPR_KCLASS_SMOOTH, (black_pre_kernel<T, false><<<nh, SB, 0, s>>>(L.lay, Pre<T>::A(L), Pre<T>::r(L),
                                                                               Pre<T>::x(L), Pre<T>::res(L))));
      if (l == 0 && k == ctx->opt.mg_post && skip_last_red) break;
      TIMED(CPR_KCLASS_SMOOTH, (red_kernel<T><<<nh, SB, 0, s>>>(L.lay, Pre<T>::A(L), Pre<T>::r(L), Pre<T>::x(L))));
    }
    // the learned correction on this level, before the finer levels'
    // post-smoothing (cpr_setup checked that it is a multi-block level)
    if (learned_on(ctx) && ctx->opt.nn_level == l && l > 0) learned_stage_at(ctx, l);
  }
}

template <int B, typename T, typename VT>
void stage2(cpr_ctx* ctx, const VT* vr, const T* z1, double* z, bool sweep, double* zn = nullptr) {
  hipStream_t s = ctx->stream;
  const Lay& L = ctx->lay;
  MGLevel& L0 = ctx->levels[0];
  const T* rp = Pre<T>::r(L0);
  T* dp = Pre<T>::x(L0);
  const T* J = Pre<T>::J(ctx);
  const T* R0 = Pre<T>::R0(ctx);
  const T* Dinv = Pre<T>::Dinv(ctx);
  T* Y = Pre<T>::Y(ctx);
  if (ctx->opt.ilu_order == CPR_ILU_TILES) {   // P-then-F only: z1 is null
    const int nt = div_up(tile_threads(L), SB);
    TIMED(CPR_KCLASS_ILU,
          (stage2_tiles_red_fwd_kernel<B, T, VT><<<nt, SB, 0, s>>>(L, J, R0, Dinv, vr, rp, dp, Y)));
    TIMED(CPR_KCLASS_ILU,
          (stage2_tiles_black_kernel<B, T, VT><<<nt, SB, 0, s>>>(L, J, R0, Dinv, vr, rp, dp, Y, z)));
    TIMED(CPR_KCLASS_ILU, (stage2_tiles_red_bwd_kernel<B, T><<<nt, SB, 0, s>>>(L, J, R0, Dinv, dp, Y, z)));
    return;
  }
  int nh = div_up(L.nh, SB);
  if (sweep)
    TIMED(CPR_KCLASS_ILU, (stage2_red_fwd_kernel<B, T, VT, true><<<nh, SB, 0, s>>>(L, J, R0, Dinv, vr, rp, dp, Y)));
  else
    TIMED(CPR_KCLASS_ILU, (stage2_red_fwd_kernel<B, T, VT, false><<<nh, SB, 0, s>>>(L, J, R0, Dinv, vr, rp, dp, Y)));
  TIMED(CPR_KCLASS_ILU, (stage2_black_kernel<B, T, VT><<<nh, SB, 0, s>>>(L, J, R0, Dinv, vr, rp, dp, Y, z1, z)));
  if (zn)
    TIMED(CPR_KCLASS_ILU, (stage2_red_bwd_kernel<B, T, true><<<nh, SB, 0, s>>>(L, J, R0, Dinv, dp, Y, z1, z, zn)));
  else
    TIMED(CPR_KCLASS_ILU, (stage2_red_bwd_kernel<B, T, false><<<nh, SB, 0, s>>>(L, J, R0, Dinv, dp, Y, z1, z, zn)));
}

template <int B, typename T, bool ABF, bool FPF>
void apply_variant(cpr_ctx* ctx, const double* vin, double* v, const double* nrm2, double* z, const double* v0,
                   const double* redc) {
  hipStream_t s = ctx->stream;
  const Lay& L = ctx->lay;
  MGLevel& L0 = ctx->levels[0];
  T* rp = Pre<T>::r(L0);
  T* x0 = Pre<T>::x(L0);
  T* Rt = Pre<T>::Rt(ctx);
  T* Z1 = Pre<T>::Z1(ctx);
  const T* J = Pre<T>::J(ctx);
  const T* R0 = Pre<T>::R0(ctx);
  const T* Dinv = Pre<T>::Dinv(ctx);
  const double* w = ABF ? ctx->Wabf : ctx->w;
  decouple_full_kernel<B, T, ABF, FPF><<<div_up(L.n, SB), SB, 0, s>>>(L.n, L.nh, w, vin, v, nrm2, v0, redc,
                                                                        Pre<T>::A(L0), Dinv, rp, x0, Rt, Z1);
  if (FPF) {
    int nh = div_up(L.nh, SB);
    TIMED(CPR_KCLASS_ILU, (fpf_black_kernel<B, T><<<nh, SB, 0, s>>>(L, J, R0, Dinv, Rt, Z1)));
    TIMED(CPR_KCLASS_ILU, (fpf_red_bwd_kernel<B, T><<<nh, SB, 0, s>>>(L, J, R0, Dinv, Z1, Rt, rp, x0)));
    TIMED(CPR_KCLASS_ILU, (fpf_resid_kernel<B, T><<<nh, SB, 0, s>>>(L, J, R0, Z1, Rt, rp)));
  }
  const bool sweep = red_sweep_in_stage2(ctx);
  vcycle<T>(ctx, sweep);
  if (learned_on(ctx) && ctx->opt.nn_level == 0) learned_stage(ctx);
  stage2<B, T, T>(ctx, Rt, FPF ? Z1 : nullptr, z, sweep);
}

// vin and z in natural order (red-black quasi-IMPES P-then-F without rate
// wells): vin is read by the first kernel alone, so z may be vin.
template <int B, typename T>
void apply_nat(cpr_ctx* ctx, const double* vin, double* z) {
  const Lay& L = ctx->lay;
  MGLevel& L0 = ctx->levels[0];
  decouple_nat_kernel<B, T><<<div_up(L.n, 256), 256, 0, ctx->stream>>>(L, ctx->w, vin, ctx->vin, Pre<T>::A(L0),
                                                                       Pre<T>::r(L0), Pre<T>::x(L0));
  const bool sweep = red_sweep_in_stage2(ctx);
  vcycle<T>(ctx, sweep);
  if (learned_on(ctx) && ctx->opt.nn_level == 0) learned_stage(ctx);
  stage2<B, T, double>(ctx, ctx->vin, nullptr, ctx->vout, sweep, z);
}

template <int B, typename T>
void apply_impl(cpr_ctx* ctx, const double* vin, double* v, const double* nrm2, double* z, const double* v0,
                const double* redc) {
  const bool abf = ctx->opt.decoupling == CPR_DECOUPLE_ABF;
  const bool fpf = ctx->opt.composition == CPR_COMPOSE_FPF;
  if (abf && fpf) return apply_variant<B, T, true, true>(ctx, vin, v, nrm2, z, v0, redc);
  if (abf) return apply_variant<B, T, true, false>(ctx, vin, v, nrm2, z, v0, redc);
  if (fpf) return apply_variant<B, T, false, true>(ctx, vin, v, nrm2, z, v0, redc);
  hipStream_t s = ctx->stream;
  const Lay& L = ctx->lay;
  MGLevel& L0 = ctx->levels[0];
  decouple_red_kernel<B, T><<<div_up(L.n, SB), SB, 0, s>>>(L.n, L.nh, ctx->w, vin, v, nrm2, v0, redc,
                                                            Pre<T>::A(L0), Pre<T>::r(L0), Pre<T>::x(L0));
  const bool sweep = red_sweep_in_stage2(ctx);
  vcycle<T>(ctx, sweep);
  if (learned_on(ctx) && ctx->opt.nn_level == 0) learned_stage(ctx);
  // rows >= 1 of the quasi-IMPES decoupled residual are those of v
  stage2<B, T, double>(ctx, v, nullptr, z, sweep);
}

}  // namespace

int vcycle_fused_level(const cpr_ctx* ctx) { return fused_level(ctx); }

// Pressure stage alone (FP64, the plain cycle even when a learned stage is
// set up): r~_p = w^T v into level 0's r, dp_mg into its x.
void precond_pressure_stage(cpr_ctx* ctx, const double* v) {
  struct PlainCycle {
    cpr_ctx* c;
    int learned;
    ~PlainCycle() { c->opt.learned = learned; }
  } plain{ctx, ctx->opt.learned};
  ctx->opt.learned = 0;
  const Lay& L = ctx->lay;
  MGLevel& L0 = ctx->levels[0];
  if (ctx->b == 1)
    decouple_red_kernel<1, double><<<div_up(L.n, SB), SB, 0, ctx->stream>>>(L.n, L.nh, ctx->w, v, nullptr, nullptr,
                                                                               nullptr, nullptr,
                                                                               L0.A, L0.r, L0.x);
  else if (ctx->b == 2)
    decouple_red_kernel<2, double><<<div_up(L.n, SB), SB, 0, ctx->stream>>>(L.n, L.nh, ctx->w, v, nullptr, nullptr,
                                                                               nullptr, nullptr,
                                                                               L0.A, L0.r, L0.x);
  else
    decouple_red_kernel<3, double><<<div_up(L.n, SB), SB, 0, ctx->stream>>>(L.n, L.nh, ctx->w, v, nullptr, nullptr,
                                                                               nullptr, nullptr,
                                                                               L0.A, L0.r, L0.x);
  vcycle<double>(ctx, false);
}

bool precond_apply_nat(cpr_ctx* ctx, const double* v, double* z) {
  if (ctx->opt.decoupling == CPR_DECOUPLE_ABF || ctx->opt.composition == CPR_COMPOSE_FPF ||
      ctx->opt.ilu_order != CPR_ILU_RED_BLACK || ctx->nrate > 0)
    return false;
  const bool mixed = precond_fp32(ctx);
  if (ctx->b == 1)
    mixed ? apply_nat<1, float>(ctx, v, z) : apply_nat<1, double>(ctx, v, z);
  else if (ctx->b == 2)
    mixed ? apply_nat<2, float>(ctx, v, z) : apply_nat<2, double>(ctx, v, z);
  else
    mixed ? apply_nat<3, float>(ctx, v, z) : apply_nat<3, double>(ctx, v, z);
  return true;
}

void precond_apply(cpr_ctx* ctx, const double* vin, double* v, const double* nrm2, double* z, const double* v0,
                   const double* redc) {
  const bool mixed = precond_fp32(ctx);
  if (ctx->b == 1) {
    if (mixed)
      apply_impl<1, float>(ctx, vin, v, nrm2, z, v0, redc);
    else
      apply_impl<1, double>(ctx, vin, v, nrm2, z, v0, redc);
  } else if (ctx->b == 2) {
    if (mixed)
      apply_impl<2, float>(ctx, vin, v, nrm2, z, v0, redc);
    else
      apply_impl<2, double>(ctx, vin, v, nrm2, z, v0, redc);
  } else {
    if (mixed)
      apply_impl<3, float>(ctx, vin, v, nrm2, z, v0, redc);
    else
      apply_impl<3, double>(ctx, vin, v, nrm2, z, v0, redc);
  }
  border_precond(ctx, vin, v, nrm2, z);   // rate wells' BHP rows, after the cell correction
}
