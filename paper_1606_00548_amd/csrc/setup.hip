// CPR preconditioner setup (Sec. 2.5: decoupling, AMG on A_pp, full-system
// smoother).
//
//  * Quasi-IMPES weights w_i = D_i^-T e_0 / (D_i^-1)_00 per cell, and row 0
//    of every decoupled block, w_i^T A_ij (the pressure equation with the
//    saturation coupling of the diagonal block removed).  A cell whose
//    (D_i^-1)_00 is zero, tiny or non-finite keeps w_i = e_0 and is counted.
//  * Pressure multigrid: A_p = (W A)_{pp}; 2x2x2 aggregation with Galerkin
//    coarse operators P^T A P, which stay 7-point; the coarsest level is
//    inverted densely (Gauss-Jordan with partial pivoting).
//  * or ABF: W_i = D_i^-1 for the diagonal block D_i, A~ = W A in full (each
//    diagonal block becomes I); a singular D_i is an error.
//  * Block ILU(0) of W A in red-then-black order: on the 7-point graph it
//    keeps every off-diagonal block and changes only the black diagonals,
//    D'_i = A~_ii - sum_k A~_ik D'_k^-1 A~_ki over the red neighbours k.
#include <algorithm>
#include <cmath>

#include "internal.h"

namespace {

constexpr double TINY = 1e-300;

// In-place inverse of a small dense matrix by Gauss-Jordan with partial
// pivoting.  Returns false for a zero, tiny or non-finite pivot.
template <int B>
__device__ bool small_inverse(double (&a)[B][B], double (&inv)[B][B]) {
  for (int r = 0; r < B; ++r)
    for (int c = 0; c < B; ++c) inv[r][c] = (r == c) ? 1.0 : 0.0;
  bool ok = true;
#pragma unroll
  for (int p = 0; p < B; ++p) {
    int piv = p;
    double best = fabs(a[p][p]);
#pragma unroll
    for (int r = p + 1; r < B; ++r)
      if (fabs(a[r][p]) > best) { best = fabs(a[r][p]); piv = r; }
    if (!(best > TINY) || !isfinite(best)) ok = false;
    if (piv != p) {
#pragma unroll
      for (int c = 0; c < B; ++c) {
        double t = a[p][c]; a[p][c] = a[piv][c]; a[piv][c] = t;
        t = inv[p][c]; inv[p][c] = inv[piv][c]; inv[piv][c] = t;
      }
    }
    double s = 1.0 / a[p][p];
#pragma unroll
    for (int c = 0; c < B; ++c) { a[p][c] *= s; inv[p][c] *= s; }
#pragma unroll
    for (int r = 0; r < B; ++r) {
      if (r == p) continue;
      double f = a[r][p];
#pragma unroll
      for (int c = 0; c < B; ++c) { a[r][c] -= f * a[p][c]; inv[r][c] -= f * inv[p][c]; }
    }
  }
  return ok;
}

// Solve D^T y = e_0 for y (small Gaussian elimination, partial pivoting).
template <int B>
__device__ bool solve_transposed_e0(const double (&D)[B][B], double (&y)[B]) {
  double a[B][B], rhs[B];
  for (int r = 0; r < B; ++r) {
    for (int c = 0; c < B; ++c) a[r][c] = D[c][r];
    rhs[r] = r == 0 ? 1.0 : 0.0;
  }
  bool ok = true;
#pragma unroll
  for (int p = 0; p < B; ++p) {
    int piv = p;
    double best = fabs(a[p][p]);
    for (int r = p + 1; r < B; ++r)
      if (fabs(a[r][p]) > best) { best = fabs(a[r][p]); piv = r; }
    if (!(best > 0.0)) ok = false;
    if (piv != p) {
      for (int c = 0; c < B; ++c) { double t = a[p][c]; a[p][c] = a[piv][c]; a[piv][c] = t; }
      double t = rhs[p]; rhs[p] = rhs[piv]; rhs[piv] = t;
    }
    for (int r = p + 1; r < B; ++r) {
      double f = a[r][p] / a[p][p];
      for (int c = p; c < B; ++c) a[r][c] -= f * a[p][c];
      rhs[r] -= f * rhs[p];
    }
  }
  for (int r = B - 1; r >= 0; --r) {
    double s = rhs[r];
    for (int c = r + 1; c < B; ++c) s -= a[r][c] * y[c];
    y[r] = s / a[r][r];
  }
  return ok;
}

template <int B, bool MIXED>
__global__ void qimpes_kernel(int n, const double* __restrict__ J, double* __restrict__ w,
                              double* __restrict__ R0, double* __restrict__ Ap, int* __restrict__ nbad,
                              float* __restrict__ Jf, float* __restrict__ Apf) {
  int t = blockIdx.x * blockDim.x + threadIdx.x;
  if (t >= n) return;
  const size_t N = n;
  double D[B][B], y[B], wv[B];
  for (int r = 0; r < B; ++r)
    for (int c = 0; c < B; ++c) D[r][c] = J[tix(7 * B * B, r * B + c, t)];
  bool ok = solve_transposed_e0<B>(D, y);
  double y0 = y[0];
  if (ok && fabs(y0) > TINY && isfinite(y0)) {
    for (int r = 0; r < B; ++r) wv[r] = y[r] / y0;
    wv[0] = 1.0;
  } else {
    for (int r = 0; r < B; ++r) wv[r] = r == 0 ? 1.0 : 0.0;
    atomicAdd(nbad, 1);
  }
  for (int r = 0; r < B; ++r) w[r * N + t] = wv[r];
  for (int d = 0; d < 7; ++d) {
    for (int c = 0; c < B; ++c) {
      double s = 0.0;
      double a[B];
      for (int r = 0; r < B; ++r) {
        a[r] = J[tix(7 * B * B, (d * B + r) * B + c, t)];
        s += wv[r] * a[r];
      }
      R0[tix(7 * B, d * B + c, t)] = s;
      if (c == 0) Ap[(size_t)d * N + t] = s;
      if (MIXED) {
        for (int r = 0; r < B; ++r) Jf[tix(7 * B * B, (d * B + r) * B + c, t)] = (float)(r == 0 ? s : a[r]);
        if (c == 0) Apf[(size_t)d * N + t] = (float)s;
      }
    }
  }
}

// ABF decoupling: W_i = D_i^-1 and A~_ij = W_i A_ij for the seven blocks of
// block row i; row 0 of every decoupled block goes to R0 (and its (0, 0)
// entry to the pressure operator), rows >= 1 to Jt.  A singular diagonal
// block raises the flag.
template <int B, bool MIXED>
__global__ void abf_kernel(int n, const double* __restrict__ J, double* __restrict__ W,
                           double* __restrict__ R0, double* __restrict__ Jt, double* __restrict__ Ap,
                           int* __restrict__ flag, float* __restrict__ Jf, float* __restrict__ Apf) {
  int t = blockIdx.x * blockDim.x + threadIdx.x;
  if (t >= n) return;
  const size_t N = n;
  double D[B][B], inv[B][B];
  for (int r = 0; r < B; ++r)
    for (int c = 0; c < B; ++c) D[r][c] = J[tix(7 * B * B, r * B + c, t)];
  if (!small_inverse<B>(D, inv)) atomicExch(flag, 1);
  for (int r = 0; r < B; ++r)
    for (int c = 0; c < B; ++c) W[((size_t)r * B + c) * N + t] = inv[r][c];
  for (int d = 0; d < 7; ++d) {
    double a[B][B];
    for (int r = 0; r < B; ++r)
      for (int c = 0; c < B; ++c) a[r][c] = J[tix(7 * B * B, (d * B + r) * B + c, t)];
    for (int r = 0; r < B; ++r)
      for (int c = 0; c < B; ++c) {
        double s = 0.0;
        for (int m = 0; m < B; ++m) s += inv[r][m] * a[m][c];
        if (r == 0) {
          R0[tix(7 * B, d * B + c, t)] = s;
          if (c == 0) Ap[(size_t)d * N + t] = s;
        } else {
          Jt[tix(7 * B * B, (d * B + r) * B + c, t)] = s;
        }
        if (MIXED) {
          Jf[tix(7 * B * B, (d * B + r) * B + c, t)] = (float)s;
          if (r == 0 && c == 0) Apf[(size_t)d * N + t] = (float)s;
        }
      }
  }
}

// Galerkin coarse operator for piecewise-constant 2x2x2 aggregation.  A
// workgroup takes 64 consecutive coarse cells in natural order and its wave
// (q, s) the fine rows (2cj+q, 2ck+s) under them, the two fine cells of its
// row per lane, so that every load of a wave is one run of 64 of a colour
// half (with eight lanes per coarse cell in storage order a load covered 16
// short runs): 26 us for 192x192x48 cells, 3.8 TB/s.  A lane sorts its cells'
// stencil rows into the coarse couplings (inside the aggregate: the diagonal);
// the partial rows are summed in a fixed order, pairs along x, then y, then z.  Ghost cells of a padded fine level take no
// part; a ghost coarse cell gets the identity row.
__global__ __launch_bounds__(256) void rap_kernel(Lay F, Lay C, const double* __restrict__ Af,
                                                  double* __restrict__ Ac, float* __restrict__ Acf) {
  __shared__ double sh[4][7][64];
  const int lane = threadIdx.x & 63, sub = threadIdx.x >> 6;
  const int cn = blockIdx.x * 64 + lane;
  double p[2][7] = {};
  int ci = 0, cj = 0, ck = 0;
  if (cn < C.n) {
    const int cjk = cn / C.nx;
    ci = cn - cjk * C.nx;
    ck = cjk / C.ny;
    cj = cjk - ck * C.ny;
    const int fj = 2 * cj + (sub & 1), fk = 2 * ck + (sub >> 1);
    if (fj < F.ny && fk < F.nz) {
      double a[2][7];
#pragma unroll
      for (int e = 0; e < 2; ++e) {
        const int f = lay_index(F, min(2 * ci + e, F.nx - 1), fj, fk);
#pragma unroll
        for (int d = 0; d < 7; ++d) a[e][d] = Af[(size_t)d * F.n + f];
      }
#pragma unroll
      for (int e = 0; e < 2; ++e) {
        const int fi = 2 * ci + e;
        if (fi >= F.nxr) continue;
        p[e][0] += a[e][0];
#pragma unroll
        for (int d = 1; d < 7; ++d) {
          int di, dj, dk;
          dir_offset(d, di, dj, dk);
          const int gi = fi + di, gj = fj + dj, gk = fk + dk;
          if (gi < 0 || gi >= F.nxr || gj < 0 || gj >= F.ny || gk < 0 || gk >= F.nz) continue;
          if ((gi >> 1) == ci && (gj >> 1) == cj && (gk >> 1) == ck)
            p[e][0] += a[e][d];
          else
            p[e][d] += a[e][d];
        }
      }
    }
  }
#pragma unroll
  for (int d = 0; d < 7; ++d) sh[sub][d][lane] = p[0][d] + p[1][d];
  __syncthreads();
  if (cn >= C.n) return;
  const int tc = lay_index(C, ci, cj, ck);
  for (int d = sub; d < 7; d += 4) {
    const double sum = (sh[0][d][lane] + sh[1][d][lane]) + (sh[2][d][lane] + sh[3][d][lane]);
    const double v = ci < C.nxr ? sum : d == 0 ? 1.0 : 0.0;
    Ac[(size_t)d * C.n + tc] = v;
    if (Acf) Acf[(size_t)d * C.n + tc] = (float)v;
  }
}

// Dense [M | I] (row-major, 2*nc columns) of the coarsest 7-point operator,
// indexed by that level's storage order.
__global__ void dense_build_kernel(Lay L, const double* __restrict__ A, double* __restrict__ M) {
  int t = blockIdx.x * blockDim.x + threadIdx.x;
  int nc = L.n;
  if (t >= nc) return;
  double* row = M + (size_t)t * 2 * nc;
  for (int c = 0; c < 2 * nc; ++c) row[c] = 0.0;
  row[nc + t] = 1.0;
  int i, j, k;
  lay_coords(L, t, i, j, k);
  row[t] += A[t];
  for (int d = 1; d < 7; ++d) {
    int nb = lay_nbr(L, i, j, k, d);
    if (nb >= 0) row[nb] += A[(size_t)d * nc + t];
  }
}

// One Gauss-Jordan column step p, double-buffered (src -> dst): every block
// finds the pivot row redundantly, then updates its share of the entries.
__global__ void gj_step_kernel(int nc, int p, const double* __restrict__ src, double* __restrict__ dst,
                               int* __restrict__ flag) {
  __shared__ double sval[256];
  __shared__ int sidx[256];
  const int w = 2 * nc;
  // pivot search over rows p..nc-1 (ties: lowest row)
  double best = -1.0;
  int bi = p;
  for (int r = p + threadIdx.x; r < nc; r += blockDim.x) {
    double v = fabs(src[(size_t)r * w + p]);
    if (v > best) { best = v; bi = r; }
  }
  sval[threadIdx.x] = best;
  sidx[threadIdx.x] = bi;
  __syncthreads();
  for (int s = blockDim.x / 2; s > 0; s >>= 1) {
    if (threadIdx.x < s) {
      double o = sval[threadIdx.x + s];
      int oi = sidx[threadIdx.x + s];
      if (o > sval[threadIdx.x] || (o == sval[threadIdx.x] && oi < sidx[threadIdx.x])) {
        sval[threadIdx.x] = o;
        sidx[threadIdx.x] = oi;
      }
    }
    __syncthreads();
  }
  int piv = sidx[0];
  double pv = src[(size_t)piv * w + p];
  if (blockIdx.x == 0 && threadIdx.x == 0 && (!(fabs(pv) > TINY) || !isfinite(pv))) atomicExch(flag, 1);
  double inv = 1.0 / pv;
  size_t total = (size_t)nc * w;
  for (size_t e = (size_t)blockIdx.x * blockDim.x + threadIdx.x; e < total;
       e += (size_t)gridDim.x * blockDim.x) {
    int r = (int)(e / w), c = (int)(e % w);
    double prow = src[(size_t)piv * w + c] * inv;   // scaled pivot row
    double out;
    if (r == p) {
      out = prow;
    } else {
      int rr = (r == piv) ? p : r;                  // row piv receives old row p
      double f = src[(size_t)rr * w + p];
      out = src[(size_t)rr * w + c] - f * prow;
    }
    dst[e] = out;
  }
}

constexpr int SCHUR_MAX = 512;   // coarsest levels up to this size are inverted through the Schur complement
// ... of those above this size, the ones whose red diagonals are no pivots by
// Gauss-Jordan over all rows (below); up to it a red diagonal of zero is an error
constexpr int SCHUR_ONLY_MAX = 128;
constexpr double PIVOT_GROWTH = 64.0;

// Coarsest inverse through the red-black Schur complement (nc <= 512).  A
// 7-point operator couples red cells only to black ones, so with the cells
// ordered red then black A = [Dr B; C Db] with diagonal Dr, Db, and
//   S = Db - C Dr^-1 B,
//   A^-1 = [Dr^-1 - X C Dr^-1, X; -S^-1 C Dr^-1, S^-1],  X = -Dr^-1 B S^-1.
// Only S (at most 256 x 256) goes through Gauss-Jordan with partial
// pivoting, in one workgroup (schur_invert_kernel); B and C have at most six
// entries per row and column, so S and the other blocks are short sums, one
// thread per entry (schur_build_kernel, schur_expand_kernel).  The red cells are
// eliminated by their diagonals, without pivoting.  A pressure operator's
// diagonal is at least about the size of its cell's couplings, but decoupled or
// imported systems need not be like that: where a multiplier (a black row's
// coupling to a red cell over that cell's diagonal) exceeds PIVOT_GROWTH, two
// decimal digits, or a red diagonal or S pivot is zero or not finite, the flag
// is set.
//
// Position of coarsest cell t among the cells of its colour: its place in
// the colour's half, or t / 2 in natural order (nx is odd there, so colours
// alternate along t within a plane, and over the whole grid or plane by
// plane with an even number of cells each).
__device__ inline int colour_pos(const Lay& L, int t) { return L.cs ? (t < L.nh ? t : t - L.nh) : t >> 1; }
// The black cell at position q.
__device__ inline int black_cell(const Lay& L, int q) {
  if (L.cs) return L.nh + q;
  int i, j, k;
  lay_coords(L, 2 * q, i, j, k);
  return 2 * q + 1 - ((i + j + k) & 1);
}
__device__ inline int colour_of(const Lay& L, int t) {
  int i, j, k;
  lay_coords(L, t, i, j, k);
  return (i + j + k) & 1;
}

// Maximum over a wavefront, to every lane: rows of 16 lanes by shifts, then
// the rows' last lanes broadcast upwards (DPP moves, a tenth of the latency
// of the same butterfly through LDS permutes).
__device__ inline unsigned wave_max(unsigned k) {
  auto step = [&](unsigned o) { k = o > k ? o : k; };
  step((unsigned)__builtin_amdgcn_update_dpp(0, (int)k, 0x111, 0xf, 0xf, false));   // row_shr:1
  step((unsigned)__builtin_amdgcn_update_dpp(0, (int)k, 0x112, 0xf, 0xf, false));
  step((unsigned)__builtin_amdgcn_update_dpp(0, (int)k, 0x114, 0xf, 0xf, false));
  step((unsigned)__builtin_amdgcn_update_dpp(0, (int)k, 0x118, 0xf, 0xf, false));
  step((unsigned)__builtin_amdgcn_update_dpp(0, (int)k, 0x142, 0xa, 0xf, false));   // row_bcast:15
  step((unsigned)__builtin_amdgcn_update_dpp(0, (int)k, 0x143, 0xc, 0xf, false));   // row_bcast:31
  return (unsigned)__builtin_amdgcn_readlane((int)k, 63);
}

// S = Db - C Dr^-1 B (row major), one thread per entry: black cells couple
// through the red cells adjacent to both.
__global__ __launch_bounds__(256) void schur_build_kernel(Lay L, const double* __restrict__ A, double* __restrict__ S,
                                                          double growth, int* __restrict__ flag) {
  const int nc = L.n, nb = L.cs ? L.nh : nc / 2;
  const int g = blockIdx.x * blockDim.x + threadIdx.x;
  if (g < nc && colour_of(L, g) == 0) {
    const double d = fabs(A[g]);
    double most = 0.0;   // of the black rows' couplings to this cell
    int i, j, k;
    lay_coords(L, g, i, j, k);
#pragma unroll
    for (int e = 0; e < 6; ++e) {
      const int n = lay_nbr(L, i, j, k, e + 1);
      if (n >= 0) most = fmax(most, fabs(A[(size_t)((e ^ 1) + 1) * nc + n]));
    }
    if (!(d > TINY) || !isfinite(d) || most > growth * d) atomicExch(flag, 1);
  }
  if (g >= nb * nb) return;
  const int t1 = black_cell(L, g / nb), t2 = black_cell(L, g % nb);
  int i, j, k, i2, j2, k2;
  lay_coords(L, t1, i, j, k);
  lay_coords(L, t2, i2, j2, k2);
  double v = t1 == t2 ? A[t1] : 0.0;
  if (abs(i - i2) + abs(j - j2) + abs(k - k2) <= 2) {
#pragma unroll
    for (int e = 1; e < 7; ++e) {
      int di, dj, dk;
      dir_offset(e, di, dj, dk);
      const int r = lay_nbr(L, i, j, k, e);
      // direction from the red cell (i + di, ...) on to t2, if they are adjacent
      const int ei = i2 - i - di, ej = j2 - j - dj, ek = k2 - k - dk;
      if (r < 0 || abs(ei) + abs(ej) + abs(ek) != 1) continue;
      const int e2 = ei ? (ei < 0 ? 1 : 2) : ej ? (ej < 0 ? 3 : 4) : (ek < 0 ? 5 : 6);
      v -= A[(size_t)e * nc + t1] * (1.0 / A[r]) * A[(size_t)e2 * nc + r];
    }
  }
  S[g] = v;
}

// S^-1 (row major, into `out`) by in-place Gauss-Jordan on nb <= NB rows.
// The pivots are a serial chain, so the matrix stays in one workgroup:
// thread (ty, tx) of TR x TC owns rows ty + TR a and columns tx + TC b, RR x
// CC entries of which CR columns' are registers (all but the largest form,
// whose 512 KB need LDS as well), and a step costs two barriers: every wave
// finds the pivot among the unused rows by itself from the column written
// last; the pivot row's owners write it out; all update, and the owners of
// the next column write that.  Rows are not exchanged: the row of pivot p is
// remembered, and the exchange form leaves M[q_p][p'] = S^-1[p][q_p'].  The
// pivot's magnitude is compared in its leading 23 bits (exponent and 12 bits
// of the mantissa, the row index below them: the lowest row of nearly equal
// ones), which bounds the multipliers by 1 + 2^-12; with EXACT in full.
// A 432-cell coarsest level (192x192x48) takes 403 us with the kernels around
// it (383 here), where one launch per column of the whole operator took 2680.
template <int NB, int TR, int TC, int CR, bool EXACT = false>
__global__ __launch_bounds__(TR * TC) void schur_invert_kernel(int nb, const double* __restrict__ S,
                                                               double* __restrict__ out, int* __restrict__ flag) {
  constexpr int NT = TR * TC, RR = NB / TR, CC = NB / TC, NS = (NB + 63) / 64;
  extern __shared__ double sm[];      // [(CC - CR) * RR][NT]
  __shared__ double col[2][NS * 64], row[NB];
  __shared__ int prow[NB], pcol[NB];
  const int tid = threadIdx.x, tx = tid % TC, ty = tid / TC, lane = tid & 63;
  double m[RR][CR];
  auto get = [&](int a, int b) -> double { return b < CR ? m[a][b < CR ? b : 0] : sm[((b - CR) * RR + a) * NT + tid]; };
  auto put = [&](int a, int b, double v) {
    if (b < CR) m[a][b < CR ? b : 0] = v; else sm[((b - CR) * RR + a) * NT + tid] = v;
  };
#pragma unroll
  for (int a = 0; a < RR; ++a)
#pragma unroll
    for (int b = 0; b < CC; ++b) {
      const int r = ty + TR * a, c = tx + TC * b;
      put(a, b, r < nb && c < nb ? S[(size_t)r * nb + c] : 0.0);
    }
  if (tx == 0)
#pragma unroll
    for (int a = 0; a < RR; ++a) col[0][ty + TR * a] = m[a][0];
  unsigned used = 0;   // bit i: row lane + 64 i is a pivot already (or none)
#pragma unroll
  for (int i = 0; i < NS; ++i)
    if (lane + 64 * i >= nb) used |= 1u << i;
  __syncthreads();
  for (int p = 0; p < nb; ++p) {
    const double* cp = col[p & 1];
    int q;
    if constexpr (EXACT) {
      static_assert(NS == 1, "a row a lane");
      double best = used ? -1.0 : fabs(cp[lane]);
      q = lane;
      for (int o = 32; o > 0; o >>= 1) {
        const double ov = __shfl_xor(best, o);
        const int oq = __shfl_xor(q, o);
        if (ov > best || (ov == best && oq < q)) {
          best = ov;
          q = oq;
        }
      }
      q = __builtin_amdgcn_readfirstlane(q);
    } else {
      unsigned key = 0;
#pragma unroll
      for (int i = 0; i < NS; ++i) {
        const int r = lane + 64 * i;
        const unsigned k = (((unsigned)__double2hiint(cp[r]) & 0x7fffff00u) | (255u - (unsigned)r)) + 1u;
        if (!((used >> i) & 1u) && k > key) key = k;
      }
      q = (int)(255u - ((wave_max(key) - 1u) & 255u));
    }
    const double pv = cp[q];
    if ((q & 63) == lane) used |= 1u << (q >> 6);
    if (tid == 0) {
      prow[p] = q;
      pcol[q] = p;
      if (!(fabs(pv) > TINY) || !isfinite(pv)) atomicExch(flag, 1);
    }
    const double pinv = 1.0 / pv;
    const int qa = q / TR;
    if (ty == q % TR) {
#pragma unroll
      for (int a = 0; a < RR; ++a)
        if (a == qa) {
#pragma unroll
          for (int b = 0; b < CC; ++b)
            row[tx + TC * b] = tx + TC * b == p ? 1.0 : get(a, b);
        }
    }
    __syncthreads();
    double f[RR];
#pragma unroll
    for (int a = 0; a < RR; ++a) f[a] = cp[ty + TR * a];
    double* cn = col[(p + 1) & 1];
    const int pb = p / TC, px = p % TC, nxb = (p + 1) / TC, nxx = (p + 1) % TC;
    if (tx == px) {   // column p starts from zero: it receives -f / pivot
#pragma unroll
      for (int b = 0; b < CC; ++b)
        if (b == pb)
#pragma unroll
          for (int a = 0; a < RR; ++a) put(a, b, 0.0);
    }
#pragma unroll
    for (int b = 0; b < CC; ++b) {
      const double pr = row[tx + TC * b] * pinv;
#pragma unroll
      for (int a = 0; a < RR; ++a) put(a, b, get(a, b) - f[a] * pr);
    }
    if (ty == q % TR) {   // the pivot row itself
#pragma unroll
      for (int a = 0; a < RR; ++a)
        if (a == qa)
#pragma unroll
          for (int b = 0; b < CC; ++b) put(a, b, row[tx + TC * b] * pinv);
    }
    if (tx == nxx) {
#pragma unroll
      for (int b = 0; b < CC; ++b)
        if (b == nxb)
#pragma unroll
          for (int a = 0; a < RR; ++a) cn[ty + TR * a] = get(a, b);
    }
    __syncthreads();
  }
#pragma unroll
  for (int b = 0; b < CC; ++b)
#pragma unroll
    for (int a = 0; a < RR; ++a) {
      const int r = ty + TR * a, c = tx + TC * b;
      if (r < nb && c < nb)
        out[(size_t)pcol[r] * nb + prow[c]] = get(a, b);
    }
}

// The same with a wavefront's lanes as the rows, for nb <= 64 RR and <= NW CC:
// lane l of wave w holds rows l + 64 i of columns CC w ..., and a step costs
// one barrier.  The pivot row is broadcast by scalar reads of its lane, and an
// entry's update is those two reads (shared by the lane's rows) and one
// multiply-add: the pivot row is not divided by its pivot until the end (a
// row's later updates are proportional to its own entries, so its scale
// factors out), which also makes its multiplier zero instead of a select.
// What passes through LDS are the pivot column's values (the multipliers) and
// the pivot's row and reciprocal; the wave that owns column p + 1 finds them
// as soon as it has updated that column, in one block of code with its other
// updates, which hide the search and the division.  The wave whose columns
// are eliminated moves them down one register a step, so that no loop needs a
// register index and all stay rolled (a step unrolled over the columns was
// bound by instruction fetch).  Sixteen waves, so that the owner's other
// updates are few: with four of sixteen columns the 64-row form took 36 us,
// with sixteen of four 31 (50 in the general form); 168 rows 214 us (296).
// Above 192 rows the entries of sixteen waves do not fit the registers, and
// eight waves are no faster than the general form.
template <int RR, int CC, int NW>
__global__ __launch_bounds__(64 * NW) __attribute__((amdgpu_waves_per_eu(NW / 4, NW / 4))) void schur_lanes_kernel(
    int nb, const double* __restrict__ S, double* __restrict__ out, int* __restrict__ flag) {
  static_assert(64 * RR <= 256 && NW * CC <= 256, "the pivot's row is kept in eight bits");
  __shared__ double col[2][RR][64], pinv_s[NW * CC];
  __shared__ int prow[NW * CC], pcol[64 * RR];
  const int lane = threadIdx.x & 63, wave = __builtin_amdgcn_readfirstlane(threadIdx.x >> 6);
  double m[CC][RR];
#pragma unroll
  for (int c = 0; c < CC; ++c)
#pragma unroll
    for (int i = 0; i < RR; ++i) {
      const int r = lane + 64 * i, cc = wave * CC + c;
      m[c][i] = r < nb && cc < nb ? S[(size_t)r * nb + cc] : 0.0;
    }
  auto bcast = [](double v, int q) {   // lane q's value to the wave
    return __hiloint2double(__builtin_amdgcn_readlane(__double2hiint(v), q),
                            __builtin_amdgcn_readlane(__double2loint(v), q));
  };
  bool used[RR], bad = false;
#pragma unroll
  for (int i = 0; i < RR; ++i) used[i] = lane + 64 * i >= nb;
  // the pivot of column p from its values v
  auto pivot = [&](int p, const double(&v)[RR]) {
    unsigned key = 0;
#pragma unroll
    for (int i = 0; i < RR; ++i) {
      const unsigned row = lane + 64 * i;
      const unsigned k = (((unsigned)__double2hiint(v[i]) & 0x7fffff00u) | (255u - row)) + 1u;
      key = used[i] || k < key ? key : k;
      col[p & 1][i][lane] = v[i];
    }
    const int q = (int)(255u - ((wave_max(key) - 1u) & 255u));   // an unused row of nb always
    double pv = bcast(v[0], q & 63);
#pragma unroll
    for (int i = 1; i < RR; ++i) pv = q >> 6 == i ? bcast(v[i], q & 63) : pv;
    bad |= !(fabs(pv) > TINY && fabs(pv) < HUGE_VAL);
    const double r = 1.0 / pv;
    if (lane == 0) {
      prow[p] = q;
      pinv_s[p] = r;
    }
  };
  double fp[RR];   // the multipliers over the pivot
  bool is_q[RR];
  int q;
  auto begin = [&](int p) {
    q = __builtin_amdgcn_readfirstlane(prow[p]);
    const double pinv = pinv_s[p];
#pragma unroll
    for (int i = 0; i < RR; ++i) {
      is_q[i] = lane + 64 * i == q;
      used[i] |= is_q[i];
      fp[i] = is_q[i] ? 0.0 : col[p & 1][i][lane] * pinv;
    }
  };
  double row[CC];   // the pivot row of this wave's columns
  auto read_row = [&] {
#pragma unroll
    for (int i = 0; i < RR; ++i)
      if (q >> 6 == i) {
#pragma unroll
        for (int c = 0; c < CC; ++c) row[c] = bcast(m[c][i], q & 63);
      }
  };
  auto pass = [&](int p) {
    begin(p);
    read_row();
#pragma unroll
    for (int c = 0; c < CC; ++c)
#pragma unroll
      for (int i = 0; i < RR; ++i) m[c][i] -= fp[i] * row[c];
  };
  auto own = [&](int p, bool more) {
    begin(p);
    read_row();
    double next[RR];
#pragma unroll
    for (int i = 0; i < RR; ++i) next[i] = m[1][i] - fp[i] * row[1];
    if (more) pivot(p + 1, next);
#pragma unroll
    for (int i = 0; i < RR; ++i) {
      m[0][i] = next[i];
#pragma unroll
      for (int c = 2; c < CC; ++c) m[c - 1][i] = m[c][i] - fp[i] * row[c];
      m[CC - 1][i] = is_q[i] ? 1.0 : -fp[i];
    }
    __syncthreads();
  };
  // the columns of the waves before this one, its own, and the others; each
  // wave passes the barrier once a column
  const int lo = min(CC * wave, nb), hi = min(lo + CC, nb);
  if (wave == 0) pivot(0, m[0]);
  __syncthreads();
  for (int p = 0; p + 1 < lo; ++p) {
    pass(p);
    __syncthreads();
  }
  if (lo > 0) {
    pass(lo - 1);
    if (lo < hi) pivot(lo, m[0]);
    __syncthreads();
  }
  for (int p = lo; p + 1 < hi; ++p) own(p, true);
  if (lo < hi) own(hi - 1, false);
  for (int p = hi; p < nb; ++p) {
    pass(p);
    __syncthreads();
  }
  for (int p = threadIdx.x; p < nb; p += 64 * NW) pcol[prow[p]] = p;
  __syncthreads();
  const int moved = hi - lo;   // register c holds column (c + moved) mod CC
#pragma unroll
  for (int i = 0; i < RR; ++i) {
    const int r = lane + 64 * i;
    if (r >= nb) continue;
    const int to = pcol[r];
    const double scale = pinv_s[to];
#pragma unroll
    for (int c = 0; c < CC; ++c) {
      const int cc = wave * CC + (c + moved < CC ? c + moved : c + moved - CC);
      if (cc < nb) out[(size_t)to * nb + prow[cc]] = m[c][i] * scale;
    }
  }
  if (bad) atomicExch(flag, 1);
}

// A^-1 (column major, and as FP32) from S^-1, one thread per entry.
__global__ __launch_bounds__(256) void schur_expand_kernel(Lay L, const double* __restrict__ A,
                                                           const double* __restrict__ Si, double* __restrict__ inv,
                                                           float* __restrict__ invf) {
  const int nc = L.n, nb = L.cs ? L.nh : nc / 2;
  const int q = blockIdx.x * blockDim.x + threadIdx.x;
  if (q >= nc * nc) return;
  const int ci = q / nc, ri = q % nc;       // column cell, row cell
  const int pc = colour_pos(L, ci), pr = colour_pos(L, ri);
  const bool rb = colour_of(L, ri) == 1, cb = colour_of(L, ci) == 1;
  int rn[6];
  double rv[6];
  {
    int i, j, k;
    lay_coords(L, ri, i, j, k);
#pragma unroll
    for (int e = 0; e < 6; ++e) {
      const int n = lay_nbr(L, i, j, k, e + 1);
      rn[e] = n >= 0 ? colour_pos(L, n) : -1;
      rv[e] = n >= 0 ? A[(size_t)(e + 1) * nc + ri] : 0.0;
    }
  }
  // (row, black column j) of A^-1
  auto black_col = [&](int j) {
    if (rb) return Si[(size_t)pr * nb + j];
    double v = 0.0;
#pragma unroll
    for (int e = 0; e < 6; ++e)
      if (rn[e] >= 0) v += rv[e] * Si[(size_t)rn[e] * nb + j];
    return -(1.0 / A[ri]) * v;
  };
  double v;
  if (cb) {
    v = black_col(pc);
  } else {
    v = 0.0;
    int i, j, k;
    lay_coords(L, ci, i, j, k);
    for (int e = 0; e < 6; ++e) {
      const int n = lay_nbr(L, i, j, k, e + 1);
      if (n >= 0) v += black_col(colour_pos(L, n)) * A[(size_t)((e ^ 1) + 1) * nc + n];
    }
    const double dc = 1.0 / A[ci];
    v = (ri == ci ? dc : 0.0) - v * dc;
  }
  inv[q] = v;
  if (invf) invf[q] = (float)v;
}

// Copy the right half of [I | M^-1] into column-major storage.
__global__ void gj_extract_kernel(int nc, const double* __restrict__ M, double* __restrict__ inv,
                                  float* __restrict__ invf) {
  int e = blockIdx.x * blockDim.x + threadIdx.x;
  if (e >= nc * nc) return;
  int col = e / nc, row = e % nc;
  double v = M[(size_t)row * 2 * nc + nc + col];
  inv[e] = v;
  if (invf) invf[e] = (float)v;
}

// Decoupled block (d, r, c) of cell t: row 0 from R0, other rows from J.
template <int B>
__device__ inline double at_blk(const double* __restrict__ J, const double* __restrict__ R0, size_t N,
                                int d, int r, int c, int t) {
  return r == 0 ? R0[tix(7 * B, d * B + c, t)] : J[tix(7 * B * B, (d * B + r) * B + c, t)];
}

template <int B>
__global__ void ilu_kernel(Lay L, int colour, const double* __restrict__ J, const double* __restrict__ R0,
                           double* __restrict__ Dinv, int* __restrict__ flag, float* __restrict__ Dinvf) {
  int q = blockIdx.x * blockDim.x + threadIdx.x;
  if (q >= L.nh) return;
  int t = colour * L.nh + q;
  const size_t N = L.n;
  double D[B][B];
  for (int r = 0; r < B; ++r)
    for (int c = 0; c < B; ++c) D[r][c] = at_blk<B>(J, R0, N, 0, r, c, t);
  if (colour == 1) {
    int i, j, k;
    lay_coords(L, t, i, j, k);
    for (int d = 1; d < 7; ++d) {
      int nb = lay_nbr(L, i, j, k, d);
      if (nb < 0) continue;
      int od = (d & 1) ? d + 1 : d - 1;   // direction from the neighbour back to t
      double Aik[B][B], Dk[B][B], Aki[B][B], T1[B][B];
      for (int r = 0; r < B; ++r)
        for (int c = 0; c < B; ++c) {
          Aik[r][c] = at_blk<B>(J, R0, N, d, r, c, t);
          Dk[r][c] = Dinv[tix(B * B, r * B + c, nb)];
          Aki[r][c] = at_blk<B>(J, R0, N, od, r, c, nb);
        }
      for (int r = 0; r < B; ++r)
        for (int c = 0; c < B; ++c) {
          double s = 0.0;
          for (int m = 0; m < B; ++m) s += Aik[r][m] * Dk[m][c];
          T1[r][c] = s;
        }
      for (int r = 0; r < B; ++r)
        for (int c = 0; c < B; ++c) {
          double s = 0.0;
          for (int m = 0; m < B; ++m) s += T1[r][m] * Aki[m][c];
          D[r][c] -= s;
        }
    }
  }
  double inv[B][B];
  if (!small_inverse<B>(D, inv)) atomicExch(flag, 1);
  for (int r = 0; r < B; ++r)
    for (int c = 0; c < B; ++c) {
      Dinv[tix(B * B, r * B + c, t)] = inv[r][c];
      if (Dinvf) Dinvf[tix(B * B, r * B + c, t)] = (float)inv[r][c];
    }
}

// Block ILU(0) diagonals in the tiled red-black order, one thread per tile
// of one colour (red tiles first): the tile's cells in order q = 0..3, each
// D'_q = A~_qq - sum over earlier neighbours k, in direction order, of
// A~_qk D'_k^-1 A~_kq.  Earlier: the tile-mates before q, and for a black
// tile every neighbour in another tile (all of them red).
template <int B>
__global__ void ilu_tiles_kernel(Lay L, int colour, const double* __restrict__ J, const double* __restrict__ R0,
                                 double* Dinv, int* __restrict__ flag, float* __restrict__ Dinvf) {
  int i, tj, tk;
  if (!tile_of_thread(L, colour, (long)blockIdx.x * blockDim.x + threadIdx.x, i, tj, tk)) return;
  const size_t N = L.n;
  for (int q = 0; q < 4; ++q) {
    const int j = 2 * tj + (q & 1), k = 2 * tk + (q >> 1);
    if (j >= L.ny || k >= L.nz) continue;
    const int t = lay_index(L, i, j, k);
    double D[B][B];
    for (int r = 0; r < B; ++r)
      for (int c = 0; c < B; ++c) D[r][c] = at_blk<B>(J, R0, N, 0, r, c, t);
    for (int d = 1; d < 7; ++d) {
      const int nb = lay_nbr(L, i, j, k, d);
      if (nb < 0) continue;
      const int mate = tile_mate(q, d);
      if (mate >= 0 ? mate > q : colour == 0) continue;   // a later neighbour
      const int od = (d & 1) ? d + 1 : d - 1;   // direction from the neighbour back to t
      double Aik[B][B], Dk[B][B], Aki[B][B], T1[B][B];
      for (int r = 0; r < B; ++r)
        for (int c = 0; c < B; ++c) {
          Aik[r][c] = at_blk<B>(J, R0, N, d, r, c, t);
          Dk[r][c] = Dinv[tix(B * B, r * B + c, nb)];
          Aki[r][c] = at_blk<B>(J, R0, N, od, r, c, nb);
        }
      for (int r = 0; r < B; ++r)
        for (int c = 0; c < B; ++c) {
          double s = 0.0;
          for (int m = 0; m < B; ++m) s += Aik[r][m] * Dk[m][c];
          T1[r][c] = s;
        }
      for (int r = 0; r < B; ++r)
        for (int c = 0; c < B; ++c) {
          double s = 0.0;
          for (int m = 0; m < B; ++m) s += T1[r][m] * Aki[m][c];
          D[r][c] -= s;
        }
    }
    double inv[B][B];
    if (!small_inverse<B>(D, inv)) atomicExch(flag, 1);
    for (int r = 0; r < B; ++r)
      for (int c = 0; c < B; ++c) {
        Dinv[tix(B * B, r * B + c, t)] = inv[r][c];
        if (Dinvf) Dinvf[tix(B * B, r * B + c, t)] = (float)inv[r][c];
      }
  }
}

// setup's flags to pinned memory (a copy to pageable memory would be staged
// by the runtime and waited for there)
__global__ void report_flags_kernel(const int* __restrict__ flag, int* __restrict__ host) {
  if (threadIdx.x < FLAGS) host[threadIdx.x] = flag[threadIdx.x];
}

__global__ void zero_int_kernel(int* p, int n) {
  int t = blockIdx.x * blockDim.x + threadIdx.x;
  if (t < n) p[t] = 0;
}

}  // namespace

static void free_levels(cpr_ctx* ctx) {
  for (size_t l = 0; l < ctx->levels.size(); ++l) {
    MGLevel& L = ctx->levels[l];
    for (void* b : {(void*)L.A, (void*)L.Af, (void*)L.x, (void*)L.r, (void*)L.xf, (void*)L.rf, (void*)L.res,
                    (void*)L.resf})
      dev_free(ctx->mem, b);
  }
  ctx->levels.clear();
  dev_free(ctx->mem, ctx->cinv); ctx->cinv = nullptr;
  dev_free(ctx->mem, ctx->cinvf); ctx->cinvf = nullptr;
  dev_free(ctx->mem, ctx->cinv64); ctx->cinv64 = nullptr;
  dev_free(ctx->mem, ctx->gj_work); ctx->gj_work = nullptr;
}

void release_hierarchy(cpr_ctx* ctx) { free_levels(ctx); }

// Level shapes: each coarse grid has ceil(n/2) cells per axis of the real
// grid above it; coarsening continues while a level has more than
// mg_coarsest real cells.  Smoothed levels are colour-split (padded with a
// ghost column when nx is odd); the coarsest is colour-split for even nx and
// natural otherwise.
static int build_hierarchy(cpr_ctx* ctx) {
  int coarsest = ctx->opt.mg_coarsest;
  std::vector<Lay> shapes;
  shapes.push_back(ctx->lay);
  while (lay_real_cells(shapes.back()) > coarsest) {
    const Lay& f = shapes.back();
    const int nx = (f.nxr + 1) / 2, ny = (f.ny + 1) / 2, nz = (f.nz + 1) / 2;
    if ((long)nx * ny * nz > coarsest)
      shapes.push_back(make_padded_lay(nx, ny, nz));
    else
      shapes.push_back(make_lay(nx, ny, nz, true));
  }
  if (shapes.back().n > 4096) return set_err(ctx, CPR_EINVAL, "coarsest level too large");
  bool same = shapes.size() == ctx->levels.size();
  for (size_t l = 0; same && l < shapes.size(); ++l)
    same = shapes[l].nx == ctx->levels[l].lay.nx && shapes[l].ny == ctx->levels[l].lay.ny &&
           shapes[l].nz == ctx->levels[l].lay.nz && shapes[l].cs == ctx->levels[l].lay.cs &&
           shapes[l].nxr == ctx->levels[l].lay.nxr;
  if (same) return CPR_OK;
  free_levels(ctx);
  ctx->levels.resize(shapes.size());
  for (size_t l = 0; l < shapes.size(); ++l) {
    MGLevel& L = ctx->levels[l];
    L.lay = shapes[l];
    size_t n = L.lay.n;
    CPR_TRY(dev_malloc(ctx->mem, (void**)&L.A, 7 * n * sizeof(double)));
    CPR_TRY(dev_malloc(ctx->mem, (void**)&L.Af, 7 * n * sizeof(float)));
    CPR_TRY(dev_malloc(ctx->mem, (void**)&L.x, n * sizeof(double)));
    CPR_TRY(dev_malloc(ctx->mem, (void**)&L.r, n * sizeof(double)));
    CPR_TRY(dev_malloc(ctx->mem, (void**)&L.xf, n * sizeof(float)));
    CPR_TRY(dev_malloc(ctx->mem, (void**)&L.rf, n * sizeof(float)));
    CPR_TRY(dev_malloc(ctx->mem, (void**)&L.res, (n / 2 + 1) * sizeof(double)));
    CPR_TRY(dev_malloc(ctx->mem, (void**)&L.resf, (n / 2 + 1) * sizeof(float)));
  }
  size_t nc = shapes.back().n;
  CPR_TRY(dev_malloc(ctx->mem, (void**)&ctx->cinv, nc * nc * sizeof(double)));
  CPR_TRY(dev_malloc(ctx->mem, (void**)&ctx->cinvf, nc * nc * sizeof(float)));
  if (nc <= SCHUR_MAX) CPR_TRY(dev_malloc(ctx->mem, (void**)&ctx->cinv64, nc * nc * sizeof(double)));
  CPR_TRY(dev_malloc(ctx->mem, (void**)&ctx->gj_work, 2 * nc * 2 * nc * sizeof(double)));
  return CPR_OK;
}

// Decoupling; MIXED: with FP32 copies of the decoupled blocks and the fine
// level.  The per-cell kernels stream the Jacobian's planes in one-wave
// workgroups.
template <int B, bool MIXED>
static void launch_decoupling(cpr_ctx* ctx) {
  const int n = ctx->lay.n, nb = div_up(n, 64);
  const MGLevel& L0 = ctx->levels[0];
  if (ctx->opt.decoupling == CPR_DECOUPLE_ABF)
    abf_kernel<B, MIXED><<<nb, 64, 0, ctx->stream>>>(n, ctx->J, ctx->Wabf, ctx->R0, ctx->Jt, L0.A, ctx->flag, ctx->Jf,
                                                     L0.Af);
  else
    qimpes_kernel<B, MIXED><<<nb, 64, 0, ctx->stream>>>(n, ctx->J, ctx->w, ctx->R0, L0.A, ctx->flag + FLAG_QIMPES,
                                                        ctx->Jf, L0.Af);
}

// Coarsest inverse by Gauss-Jordan with partial pivoting over all rows, one
// launch a column.
static void launch_pivoted_inverse(cpr_ctx* ctx, double* inv, float* invf) {
  hipStream_t s = ctx->stream;
  const MGLevel& last = ctx->levels.back();
  const int nc = last.lay.n;
  double* bufA = ctx->gj_work;
  double* bufB = ctx->gj_work + (size_t)nc * 2 * nc;
  dense_build_kernel<<<div_up(nc, 256), 256, 0, s>>>(last.lay, last.A, bufA);
  int gblocks = div_up((long)nc * 2 * nc, 256);
  if (gblocks > 512) gblocks = 512;
  for (int p = 0; p < nc; ++p) {
    gj_step_kernel<<<gblocks, 256, 0, s>>>(nc, p, bufA, bufB, ctx->flag);
    double* t = bufA; bufA = bufB; bufB = t;
  }
  gj_extract_kernel<<<div_up((long)nc * nc, 256), 256, 0, s>>>(nc, bufA, inv, invf);
}

// The inverse that a mixed solve's FP64 fallback applies.  A system on which
// the FP32 preconditioner stalls amplifies last bits (a digit in the last place
// of the coarsest solve became 1e-5 of dx after 75 iterations), so from there
// on the solve keeps the arithmetic of one elimination for good, whichever is
// the fastest: partial pivoting over all rows, for levels of up to 128 cells
// over those of the Schur complement.  Formed by the first fallback after a
// setup.
int fallback_inverse(cpr_ctx* ctx) {
  const MGLevel& last = ctx->levels.back();
  const int nc = last.lay.n;
  if (nc > SCHUR_MAX || ctx->cinv64_done) return CPR_OK;   // setup's own is that one
  hipStream_t s = ctx->stream;
  if (nc <= SCHUR_ONLY_MAX) {
    const int nb = last.lay.cs ? last.lay.nh : nc / 2;
    double* sb = ctx->gj_work;
    double* si = ctx->gj_work + (size_t)nb * nb;
    schur_build_kernel<<<div_up(std::max(nc, nb * nb), 256), 256, 0, s>>>(last.lay, last.A, sb, HUGE_VAL,
                                                                         ctx->flag + FLAG_SINGULAR);
    if (nb > 0)
      schur_invert_kernel<64, 32, 16, 4, true><<<1, 512, 0, s>>>(nb, sb, si, ctx->flag + FLAG_SINGULAR);
    schur_expand_kernel<<<div_up((long)nc * nc, 256), 256, 0, s>>>(last.lay, last.A, si, ctx->cinv64, nullptr);
  } else {
    launch_pivoted_inverse(ctx, ctx->cinv64, nullptr);
  }
  ctx->cinv64_done = true;
  return launch_check(ctx, "coarsest inverse of the FP64 fallback");
}

// setup's flags, once its kernels have run.  Syncs.
static int read_flags(cpr_ctx* ctx, int (&flag)[FLAGS]) {
  report_flags_kernel<<<1, 64, 0, ctx->stream>>>(ctx->flag, reinterpret_cast<int*>(ctx->hhost_dev + 8));
  CPR_TRY(hipGetLastError());
  CPR_TRY(hipStreamSynchronize(ctx->stream));
  for (int q = 0; q < FLAGS; ++q) flag[q] = reinterpret_cast<const int*>(ctx->hhost + 8)[q];
  return CPR_OK;
}

int setup_cpr(cpr_ctx* ctx) {
  int rc = build_hierarchy(ctx);
  if (rc != CPR_OK) return rc;
  ctx->cinv64_done = false;
  hipStream_t s = ctx->stream;
  const Lay& L = ctx->lay;
  const int n = L.n;
  zero_int_kernel<<<1, 64, 0, s>>>(ctx->flag, FLAGS);   // and the counters of the Krylov kernels' last workgroups
  // The FP32 copies of a mixed preconditioner (decoupled blocks, levels, ILU
  // diagonals) are stored by the kernels that form the values: passes of their
  // own read them again (256x256x64 black oil: 625 us of the decoupling and
  // 680 + 95 us of the copies, 870 us together).
  const bool mixed = ctx->opt.precision == CPR_PREC_MIXED;
  float* df = mixed ? ctx->Dinvf : nullptr;
  const bool abf = ctx->opt.decoupling == CPR_DECOUPLE_ABF;
  if (ctx->b == 1)
    mixed ? launch_decoupling<1, true>(ctx) : launch_decoupling<1, false>(ctx);
  else if (ctx->b == 2)
    mixed ? launch_decoupling<2, true>(ctx) : launch_decoupling<2, false>(ctx);
  else
    mixed ? launch_decoupling<3, true>(ctx) : launch_decoupling<3, false>(ctx);
  // rows >= 1 of the decoupled blocks: the Jacobian's own (quasi-IMPES) or D^-1 A (ABF)
  const double* Jdec = abf ? ctx->Jt : ctx->J;
  // Galerkin chain and coarsest inverse, the longer chain for small systems,
  // on the caller's stream, where nothing waits for an event (Newton step of
  // 32x32x8: 852 -> 833 us).  The ILU factorisation on the auxiliary stream
  // overlaps the inverse only, a serial chain in one workgroup: its kernels
  // flood the chip, so that the Galerkin kernels beside them took as long as
  // it did and the inverse's workgroup got its place when they had drained
  // (192x192x48: 288 against 26 us and the inverse done 970 against 450 us
  // after the decoupling).
  for (size_t l = 0; l + 1 < ctx->levels.size(); ++l) {
    const MGLevel& F = ctx->levels[l];
    MGLevel& C = ctx->levels[l + 1];
    rap_kernel<<<div_up(C.lay.n, 64), 256, 0, s>>>(F.lay, C.lay, F.A, C.A, mixed ? C.Af : nullptr);
  }
  // dense inverse of the coarsest level
  const MGLevel& last = ctx->levels.back();
  int nc = last.lay.n;
  if (nc <= SCHUR_MAX) {
    const int nb = last.lay.cs ? last.lay.nh : nc / 2;
    double* sb = ctx->gj_work;
    double* si = ctx->gj_work + (size_t)nb * nb;
    const bool only = nc <= SCHUR_ONLY_MAX;
    int* bad = ctx->flag + (only ? FLAG_SINGULAR : FLAG_PIVOT);
    schur_build_kernel<<<div_up(std::max(nc, nb * nb), 256), 256, 0, s>>>(last.lay, last.A, sb,
                                                                         only ? HUGE_VAL : PIVOT_GROWTH, bad);
    CPR_TRY(hipEventRecord(ctx->ev_rap, s));
    if (nb == 0) {
      // a single, red cell: nothing to invert, schur_expand_kernel forms 1 / A
    } else if (nb <= 64) {
      schur_lanes_kernel<1, 4, 16><<<1, 1024, 0, s>>>(nb, sb, si, bad);
    } else if (nb <= 128) {
      schur_lanes_kernel<2, 8, 16><<<1, 1024, 0, s>>>(nb, sb, si, bad);
    } else if (nb <= 192) {
      schur_lanes_kernel<3, 12, 16><<<1, 1024, 0, s>>>(nb, sb, si, bad);
    } else if (nb <= 224) {
      schur_invert_kernel<224, 32, 16, 14><<<1, 512, 0, s>>>(nb, sb, si, bad);
    } else {
      constexpr int lds = 4 * 8 * 512 * sizeof(double);   // a quarter of the 256 x 256 matrix
      CPR_TRY(hipFuncSetAttribute((const void*)schur_invert_kernel<256, 32, 16, 12>,
                                  hipFuncAttributeMaxDynamicSharedMemorySize, lds));
      schur_invert_kernel<256, 32, 16, 12><<<1, 512, lds, s>>>(nb, sb, si, bad);
    }
    schur_expand_kernel<<<div_up((long)nc * nc, 256), 256, 0, s>>>(last.lay, last.A, si, ctx->cinv, ctx->cinvf);
  } else {
    CPR_TRY(hipEventRecord(ctx->ev_rap, s));
    launch_pivoted_inverse(ctx, ctx->cinv, ctx->cinvf);
  }
  hipStream_t a = ctx->aux;
  CPR_TRY(hipStreamWaitEvent(a, ctx->ev_rap, 0));
  // block ILU(0): red diagonals (cells or tiles) first, black ones use them
  const bool tiles = ctx->opt.ilu_order == CPR_ILU_TILES;
  const int nh = tiles ? (int)div_up(tile_threads(L), 64) : div_up(L.nh, 64);
  for (int colour = 0; colour < 2; ++colour) {
    if (tiles) {
      if (ctx->b == 1)
        ilu_tiles_kernel<1><<<nh, 64, 0, a>>>(L, colour, Jdec, ctx->R0, ctx->Dinv, ctx->flag, df);
      else if (ctx->b == 2)
        ilu_tiles_kernel<2><<<nh, 64, 0, a>>>(L, colour, Jdec, ctx->R0, ctx->Dinv, ctx->flag, df);
      else
        ilu_tiles_kernel<3><<<nh, 64, 0, a>>>(L, colour, Jdec, ctx->R0, ctx->Dinv, ctx->flag, df);
    } else if (ctx->b == 1) {
      ilu_kernel<1><<<nh, 64, 0, a>>>(L, colour, Jdec, ctx->R0, ctx->Dinv, ctx->flag, df);
    } else if (ctx->b == 2) {
      ilu_kernel<2><<<nh, 64, 0, a>>>(L, colour, Jdec, ctx->R0, ctx->Dinv, ctx->flag, df);
    } else {
      ilu_kernel<3><<<nh, 64, 0, a>>>(L, colour, Jdec, ctx->R0, ctx->Dinv, ctx->flag, df);
    }
  }
  CPR_TRY(hipEventRecord(ctx->ev_ilu, a));
  CPR_TRY(hipStreamWaitEvent(s, ctx->ev_ilu, 0));
  rc = launch_check(ctx, "cpr_setup kernels");
  if (rc != CPR_OK) return rc;
  int flag[FLAGS];
  if ((rc = read_flags(ctx, flag)) != CPR_OK) return rc;
  if (flag[FLAG_PIVOT] && !flag[FLAG_SINGULAR]) {
    launch_pivoted_inverse(ctx, ctx->cinv, ctx->cinvf);
    if ((rc = launch_check(ctx, "cpr_setup kernels")) != CPR_OK) return rc;
    if ((rc = read_flags(ctx, flag)) != CPR_OK) return rc;
  }
  ctx->qimpes_bad = flag[FLAG_QIMPES];
  if (flag[FLAG_SINGULAR]) return set_err(ctx, CPR_ESINGULAR, "singular ILU diagonal block or coarsest operator");
  ctx->setup_done = 1;
  return CPR_OK;
}
