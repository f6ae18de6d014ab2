// Pressure-correction network: training and inference kernels.
//
// The network (no counterpart in the paper; it supplies a correction to
// the pressure stage of the CPR preconditioner) is a 3-D U-Net on
// channels-last FP32 tensors T[b][voxel][c] (voxel = x + nx*(y + ny*z)):
//   e0 = relu(c0(x))            e1 = relu(c1(pool e0))
//   e2 = relu(c2(pool e1))      e3 = relu(c3(pool e2))
//   d2 = relu(c4(up e3)) + e2   d1 = relu(c5(up d2)) + e1
//   d0 = relu(c6(up d1)) + e0   y  = wo . d0 + bo
// with 3x3x3 zero-padded correlations, 2x2x2 average pooling, nearest
// upsampling (read on the fly by the convolution that consumes it), and a
// normalised mean-squared-error loss.  Parameters: FP32 master copy, Adam
// moments, BF16 copies laid out as MFMA fragments.
//
// Convolutions are implicit GEMMs on the CDNA matrix cores
// (v_mfma_f32_16x16x32_bf16, FP32 accumulation): M = output channels, N =
// voxels, K = 27 taps x input channels in steps of 32; activations are
// converted to BF16 as they are staged in LDS.  The data gradient is the same
// kernel with mirrored taps and transposed channel blocks; the weight gradient
// is a GEMM over voxels (M = input channels, N = output channels) whose
// per-workgroup partial sums are reduced in a fixed order, so training is
// deterministic.
#include <cmath>
#include <cstring>

#include "internal.h"

typedef __bf16 bf16x8 __attribute__((ext_vector_type(8)));
typedef float f32x4 __attribute__((ext_vector_type(4)));

namespace {

constexpr int NCONV = 7;
constexpr int CIN[NCONV] = {3, 16, 32, 64, 64, 64, 32};
constexpr int COUT[NCONV] = {16, 32, 64, 64, 64, 32, 16};
constexpr int CIN_PAD[NCONV] = {16, 16, 32, 64, 64, 64, 32};
constexpr int WG_MAX = 512;      // workgroups of one weight gradient

// FP32 -> BF16, round to nearest even (one value; staging converts pairs
// with pack_bf16x2)
__device__ inline short f2bf(float f) {
  unsigned u = __float_as_uint(f);
  u += 0x7FFFu + ((u >> 16) & 1u);
  return (short)(u >> 16);
}

typedef __bf16 bf16x2_v __attribute__((ext_vector_type(2)));
typedef float f32x2_v __attribute__((ext_vector_type(2)));

struct Geo {
  int nx, ny, nz, V;   // grid of the tensor being produced
  int batch;
};

// ------------------------------------------------------------ convolution
// out[b][v][co] = sum_t sum_ci X~[b][v + off_t][ci] W[t][ci][co]; X~ is X on
// the same grid, or X on the half-resolution grid read at (x/2, y/2, z/2)
// when UP.  EPI 1: a = relu(acc + bias), stored in outA when given, and
// a + skip stored in outD when skip is given; with head (inference only) the
// 1x1x1 head is applied to a + skip and only y is stored.  EPI 0: raw acc in
// outA (data gradient).
//
// Implicit GEMM on v_mfma_f32_16x16x32_bf16: M = output channels, N = voxels,
// K = (tap, input channel) in steps of 32, so that a lane of a result holds
// four consecutive channels of one voxel and biases, skips, activations and
// pools move as 16-byte values.  A workgroup (4 waves) owns CO/NS of the
// output channels, whose weight fragments it stages in LDS once, and with
// KS = 1 several tiles of 16 x 4 x 4 output voxels one after the other (as
// many workgroups as the chip holds).  Of a tile it stages the input (tile
// plus a one-voxel halo, or the half-resolution cells under it when UP) in
// LDS as BF16; the next tile's loads are in flight during the K loop, which
// touches LDS only (with one tile per workgroup the loads' and the weights'
// latency stood before every K loop: one sample of 128x128x64, the convolution
// at full resolution 59 -> 33 us, all seven 170 -> 128 us).
// Each wave owns one z-plane of the tile (4 N-blocks of 16 voxels along x)
// and every K-step; with KS = 4 (small grids, to keep enough waves in flight)
// the workgroup has one tile of one plane and the waves split the K-steps
// round-robin, their partial tiles summed in LDS in wave order, so results
// are deterministic either way.  POOL (KS = 1 only): the workgroup also
// writes the 2x2x2 average of its activations, which its tile holds whole.
//
// K ordering (must match frag_kernel): CI >= 32: step = t * (CI/32) + chunk,
// 32 channels per step; CI = 16: step s covers taps 2s, 2s+1; CI = 4 (the
// 3-channel input, padded): step s covers taps 8s..8s+7, 4 channels each.
// Taps past 26 have zero weights.
constexpr int TX = 16, TY = 4;

__host__ __device__ constexpr int ksteps(int ci) { return ci >= 32 ? 27 * (ci / 32) : (ci == 16 ? 14 : 4); }

// a in the low half, b in the high half, both rounded to nearest even by
// one v_cvt_pk_bf16_f32
__device__ inline unsigned pack_bf16x2(float a, float b) {
  return __builtin_bit_cast(unsigned, __builtin_convertvector(f32x2_v{a, b}, bf16x2_v));
}

struct ConvArgs {
  Geo g;
  const float* X;        // input [batch][voxel][CSRC] (half-resolution grid when UP)
  const bf16x8* W;       // all weight fragments [NK][CO/16][64]
  const float* bias;     // [CO] (EPI 1)
  const float* skip;     // [batch][voxel][CO] or null
  float* outA;           // EPI 1: relu(acc + bias) (null: not stored); EPI 0: acc
  float* outD;           // EPI 1 with skip: relu(acc + bias) + skip
  const float* head;     // fused 1x1x1 head [CO + 1] (CO = 16, KS = 1) or null
  float* y;              // head output [batch][voxel]
  float* pool;           // POOL: [batch][coarse voxel][CO]
  const double* xscale;  // CSRC = 3: device scalar multiplying input channel 2 as it is loaded, or null
};

template <int CI, bool UP, int KS>
struct ConvTile {
  static constexpr int TZ = 4 / KS;
  static constexpr int HX = UP ? TX / 2 + 2 : TX + 2, HY = UP ? TY / 2 + 2 : TY + 2, HZ = UP ? TZ / 2 + 2 : TZ + 2;
  static constexpr int HV = HX * HY * HZ;
  // halo voxel stride in bytes: padded by 16 bytes for CI >= 16 so that 16
  // lanes reading 16 bytes of 16 neighbouring voxels hit distinct banks
  static constexpr int VB = (CI >= 16 ? CI + 8 : CI) * 2;
};
template <int CI, int CO, bool UP, int KS, int NS>
__host__ __device__ constexpr int conv_lds() {
  constexpr int main = ConvTile<CI, UP, KS>::HV * ConvTile<CI, UP, KS>::VB + ksteps(CI) * (CO / NS) * 64;
  constexpr int red = KS > 1 ? KS * 64 * (CO / NS) * 4 : 0;
  return main > red ? main : red;
}
// workgroups a CU holds of a convolution that walks over tiles
constexpr int CUS = 256, CU_LDS = 160 * 1024;
template <int CI, int CO, bool UP, int KS, int NS>
__host__ __device__ constexpr int conv_per_cu() {
  constexpr int fit = CU_LDS / conv_lds<CI, CO, UP, KS, NS>();
  return KS > 1 ? 1 : fit < 4 ? fit : 4;
}

template <int CI, int CSRC, int CO, bool UP, int EPI, int KS, int NS, bool POOL>
__global__ __launch_bounds__(256, (conv_per_cu<CI, CO, UP, KS, NS>())) void conv_kernel(ConvArgs p) {
  static_assert(KS == 1 || KS == 4, "K split is 1 or 4");
  static_assert(CI == 4 || CI == 16 || CI % 32 == 0, "channel layout");
  static_assert(CO % (16 * NS) == 0, "channel split");
  static_assert(!POOL || KS == 1, "pooling needs whole 2x2x2 cells in the tile");
  using Tile = ConvTile<CI, UP, KS>;
  constexpr int TZ = Tile::TZ, HX = Tile::HX, HY = Tile::HY, HV = Tile::HV, VB = Tile::VB;
  constexpr int NK = ksteps(CI);
  constexpr int NT = CO / 16;          // M-blocks of the whole convolution
  constexpr int COB = CO / NS;         // output channels of this workgroup
  constexpr int NTB = COB / 16;
  constexpr int HALO_BYTES = HV * VB;
  static_assert(HALO_BYTES % 16 == 0 && (!POOL || 64 * COB * 4 <= HALO_BYTES), "pool sums reuse the halo");
  __shared__ __align__(16) unsigned char smem[conv_lds<CI, CO, UP, KS, NS>()];
  const bf16x8* wl = (const bf16x8*)(smem + HALO_BYTES);
  const Geo& g = p.g;

  // channel block and tiles of this workgroup; consecutive ones go to the
  // same XCD, and the channel blocks of a tile are neighbours
  const int ntx = (g.nx + TX - 1) / TX, nty = (g.ny + TY - 1) / TY, ntz = (g.nz + TZ - 1) / TZ;
  const int ntiles = ntx * nty * ntz * g.batch;
  int blk = blockIdx.x;
  if ((gridDim.x & 7) == 0) blk = (blockIdx.x & 7) * (gridDim.x >> 3) + (blockIdx.x >> 3);
  const int nb = blk % NS, walkers = gridDim.x / NS;
  const int tile0 = (int)((long)(blk / NS) * ntiles / walkers), tile1 = (int)((long)(blk / NS + 1) * ntiles / walkers);
  int x0, y0, z0, b;
  auto locate = [&](int tile) {
    x0 = tile % ntx * TX;
    y0 = (tile / ntx) % nty * TY;
    z0 = (tile / (ntx * nty)) % ntz * TZ;
    b = tile / (ntx * nty * ntz);
  };

  const int sx = UP ? g.nx >> 1 : g.nx, sy = UP ? g.ny >> 1 : g.ny, sz = UP ? g.nz >> 1 : g.nz;
  const float xs2 = (CSRC != CI && p.xscale) ? (float)*p.xscale : 1.f;
  constexpr int NQ = HV * (CI / 4), NU = (NQ + 255) / 256;
  // the input window of a tile, NU quads of channels per thread (zero outside
  // the grid)
  auto fetch = [&](float4(&v)[NU]) {
    const int ox = UP ? (x0 - 1) >> 1 : x0 - 1, oy = UP ? (y0 - 1) >> 1 : y0 - 1, oz = UP ? (z0 - 1) >> 1 : z0 - 1;
    const float* Xb = p.X + (long)b * sx * sy * sz * CSRC;
#pragma unroll
    for (int u = 0; u < NU; ++u) {
      const int q = u * 256 + threadIdx.x;
      v[u] = make_float4(0.f, 0.f, 0.f, 0.f);
      if (q < NQ) {
        const int hv = q / (CI / 4), c4 = (q % (CI / 4)) * 4;
        const int hx = hv % HX, hy = (hv / HX) % HY, hz = hv / (HX * HY);
        const int px = ox + hx, py = oy + hy, pz = oz + hz;
        if (px >= 0 && px < sx && py >= 0 && py < sy && pz >= 0 && pz < sz) {
          const float* src = Xb + ((long)px + (long)sx * (py + (long)sy * pz)) * CSRC + c4;
          if (CSRC == CI) {
            v[u] = *(const float4*)src;
          } else {
            v[u].x = src[0]; v[u].y = src[1]; v[u].z = src[2];
            v[u].w = 1.f;   // inside the grid (the fourth channel is padding)
          }
        }
      }
    }
  };
  auto place = [&](const float4(&v)[NU]) {   // the same as BF16 into LDS
#pragma unroll
    for (int u = 0; u < NU; ++u) {
      const int q = u * 256 + threadIdx.x;
      const float z = CSRC == CI ? v[u].z : v[u].w != 0.f ? v[u].z * xs2 : 0.f;
      const float w = CSRC == CI ? v[u].w : 0.f;
      if (q < NQ)
        *(uint2*)(smem + (size_t)(q / (CI / 4)) * VB + (q % (CI / 4)) * 8) =
            make_uint2(pack_bf16x2(v[u].x, v[u].y), pack_bf16x2(z, w));
    }
  };
  // a tile's quads (at most 21 a thread) are loaded a tile ahead, those of the
  // first together with the weights (at most 14 fragments a thread): one
  // round trip to memory before the first K loop
  float4 v[NU];
  locate(tile0);
  if (tile0 < tile1) fetch(v);
  {
    constexpr int NWF = NK * NTB * 64, WU = (NWF + 255) / 256;
    bf16x8 w[WU];
#pragma unroll
    for (int u = 0; u < WU; ++u) {
      const int q = u * 256 + threadIdx.x;
      if (q < NWF) {
        const int ks = q / (NTB * 64), j = (q / 64) % NTB, lane = q % 64;
        w[u] = p.W[((size_t)ks * NT + nb * NTB + j) * 64 + lane];
      }
    }
#pragma unroll
    for (int u = 0; u < WU; ++u) {
      const int q = u * 256 + threadIdx.x;
      if (q < NWF) ((bf16x8*)(smem + HALO_BYTES))[q] = w[u];
    }
  }

  const int wave = __builtin_amdgcn_readfirstlane(threadIdx.x >> 6);   // uniform: the K split branches on it
  const int lane = threadIdx.x & 63, i16 = lane & 15, kq = lane >> 4;
  const int lz = KS == 1 ? wave : 0;
  const long V = g.V;
  const int c0 = nb * COB + 4 * kq;   // first channel of this lane in M-block 0
  float4 bias[NTB] = {};
  if constexpr (EPI == 1) {
#pragma unroll
    for (int n = 0; n < NTB; ++n)
      bias[n] = make_float4(p.bias[c0 + n * 16], p.bias[c0 + n * 16 + 1], p.bias[c0 + n * 16 + 2],
                            p.bias[c0 + n * 16 + 3]);
  }

  for (int tile = tile0; tile < tile1; ++tile) {
    if (tile > tile0) __syncthreads();   // the tile before no longer needs the halo
    place(v);
    __syncthreads();

    // Byte address in the halo of the input under output voxel (i16, m, lz)
    // at tap (dx, dy, dz) = per-lane part + a part known at compile time once
    // the K loop is unrolled (folded into the LDS instructions' offsets).
    // Same grid: (i16 + 1 + dx) + HX (m + 1 + dy) + HX HY (lz + 1 + dz).
    // UP (x0, y0 multiples of 16 and 4): ((i16 + dx) >> 1) + 1 along x,
    // ((m + dy) >> 1) + 1 along y, and ((z0 + lz + dz) >> 1) - ((z0 - 1) >> 1)
    // along z, which depends on z0 and is uniform over the wave.
    const int lane_chunk = CI >= 32 ? 16 * kq : (CI == 16 ? 16 * (kq & 1) : 0);
    int base = 0;            // same grid
    int upb[3][3] = {};      // UP: [dx + 1][dz + 1]
    if constexpr (UP) {
      const int oz = (z0 - 1) >> 1;
#pragma unroll
      for (int ddx = 0; ddx < 3; ++ddx)
#pragma unroll
        for (int ddz = 0; ddz < 3; ++ddz) {
          const int zc = ((z0 + lz + ddz - 1) >> 1) - oz;
          upb[ddx][ddz] = ((((i16 + ddx - 1) >> 1) + 1) + HX * HY * zc) * VB + lane_chunk;
        }
    } else {
      base = ((i16 + 1) + HX + HX * HY * (lz + 1)) * VB + lane_chunk;
    }
    // this lane's outputs: voxel (x, y0 + m, z), channels c0 + 16 n ...
    const int x = x0 + i16, z = z0 + lz, ty = y0;
    const long o0 = (long)b * V + x + (long)g.nx * (ty + (long)g.ny * z);
    const bool oxz = x < g.nx && z < g.nz;
    // KS = 1 with a skip input: its values are loaded before the K loop so
    // that their latency hides behind the MFMAs
    float4 skv[KS == 1 && EPI == 1 ? 4 : 1][NTB];
    if constexpr (KS == 1 && EPI == 1) {
      const bool has_skip = p.skip != nullptr;
#pragma unroll
      for (int m = 0; m < 4; ++m)
#pragma unroll
        for (int n = 0; n < NTB; ++n)
          skv[m][n] = has_skip && oxz && ty + m < g.ny
                          ? *(const float4*)(p.skip + (o0 + (long)m * g.nx) * CO + c0 + n * 16)
                          : make_float4(0.f, 0.f, 0.f, 0.f);
    }
    const int tx0 = x0, tz0 = z0, tb = b;
    if (tile + 1 < tile1) {
      locate(tile + 1);
      fetch(v);
    }
    f32x4 acc[4][NTB];
#pragma unroll
    for (int m = 0; m < 4; ++m)
#pragma unroll
      for (int n = 0; n < NTB; ++n) acc[m][n] = f32x4{0.f, 0.f, 0.f, 0.f};
    // same-grid tap offset (bytes) relative to base, m = 0
    auto toff = [](int t) { return ((t % 3 - 1) + HX * ((t / 3) % 3 - 1) + HX * HY * (t / 9 - 1)) * VB; };
    if constexpr (CI >= 32) {
      // K-steps grouped by (dz, dx, channel chunk): the three dy taps of a
      // group read the same input rows, so the wave loads each row's voxel
      // fragment once (6 rows of the tile plus halo, or 4 half-resolution
      // rows when UP) and the three weight fragments, then issues 12 MFMA per
      // M-block.  Groups are split over the waves when KS = 4.
      constexpr int NCH = CI / 32;
      constexpr int NR = UP ? 4 : 6;
      auto group = [&](int kc, int dx, int dz, int row0) {   // row0: address of the first row
        bf16x8 bw[3][NTB];
#pragma unroll
        for (int ddy = 0; ddy < 3; ++ddy)
#pragma unroll
          for (int n = 0; n < NTB; ++n)
            bw[ddy][n] = wl[(((dz + 1) * 9 + ddy * 3 + (dx + 1)) * NCH + kc) * NTB * 64 + n * 64 + lane];
        bf16x8 ar[NR];
#pragma unroll
        for (int yy = 0; yy < NR; ++yy)
          ar[yy] = __builtin_bit_cast(bf16x8, *(const uint4*)(smem + row0 + HX * yy * VB + kc * 64));
#pragma unroll
        for (int ddy = 0; ddy < 3; ++ddy)
#pragma unroll
          for (int m = 0; m < 4; ++m) {
            const int yy = UP ? ((m + ddy - 1) >> 1) + 1 : m + ddy;
#pragma unroll
            for (int n = 0; n < NTB; ++n)
              acc[m][n] = __builtin_amdgcn_mfma_f32_16x16x32_bf16(bw[ddy][n], ar[yy], acc[m][n], 0, 0, 0);
          }
      };
      if constexpr (KS == 1) {
#pragma unroll
        for (int grp = 0; grp < 9 * NCH; ++grp) {
          const int kc = grp % NCH, dx = (grp / NCH) % 3 - 1, dz = grp / (3 * NCH) - 1;
          group(kc, dx, dz, UP ? upb[dx + 1][dz + 1] : base + (dx + HX * HY * dz - HX) * VB);
        }
      } else {
        // rolled: a wave runs every fourth group once, so that unrolled code
        // would be fetched for each of them
        for (int grp = wave; grp < 9 * NCH; grp += KS) {
          const int kc = grp % NCH, dx = (grp / NCH) % 3 - 1, dz = grp / (3 * NCH) - 1;
          const int up = ((((i16 + dx) >> 1) + 1) + HX * HY * (((tz0 + dz) >> 1) - ((tz0 - 1) >> 1))) * VB + lane_chunk;
          group(kc, dx, dz, UP ? up : base + (dx + HX * HY * dz - HX) * VB);
        }
      }
    } else {
#pragma unroll
      for (int ks = 0; ks < NK; ++ks) {
        if (KS > 1 && (ks % KS) != wave) continue;
        bf16x8 bw[NTB];
#pragma unroll
        for (int n = 0; n < NTB; ++n) bw[n] = wl[((size_t)ks * NTB + n) * 64 + lane];
        int sel0 = 0, sel1 = 0;     // per-lane tap offsets of this step
        if constexpr (CI == 16) {
          sel0 = (kq >> 1) ? toff(min(2 * ks + 1, 26)) : toff(2 * ks);
        } else {
          const int ta[4] = {min(8 * ks, 26), min(8 * ks + 2, 26), min(8 * ks + 4, 26), min(8 * ks + 6, 26)};
          const int tb4[4] = {min(8 * ks + 1, 26), min(8 * ks + 3, 26), min(8 * ks + 5, 26), min(8 * ks + 7, 26)};
          sel0 = kq == 0 ? toff(ta[0]) : kq == 1 ? toff(ta[1]) : kq == 2 ? toff(ta[2]) : toff(ta[3]);
          sel1 = kq == 0 ? toff(tb4[0]) : kq == 1 ? toff(tb4[1]) : kq == 2 ? toff(tb4[2]) : toff(tb4[3]);
        }
#pragma unroll
        for (int m = 0; m < 4; ++m) {
          uint4 raw;
          if constexpr (CI == 16) {
            raw = *(const uint4*)(smem + base + sel0 + HX * m * VB);
          } else {
            const uint2 lo = *(const uint2*)(smem + base + sel0 + HX * m * VB);
            const uint2 hi = *(const uint2*)(smem + base + sel1 + HX * m * VB);
            raw = make_uint4(lo.x, lo.y, hi.x, hi.y);
          }
          const bf16x8 a = __builtin_bit_cast(bf16x8, raw);
#pragma unroll
          for (int n = 0; n < NTB; ++n)
            acc[m][n] = __builtin_amdgcn_mfma_f32_16x16x32_bf16(bw[n], a, acc[m][n], 0, 0, 0);
        }
      }
    }

    if constexpr (KS == 1) {
#pragma unroll
      for (int m = 0; m < 4; ++m) {
        const bool ok = oxz && ty + m < g.ny;
        const long o = o0 + (long)m * g.nx;
        if constexpr (EPI == 1 && CO == 16) {
          if (p.head) {
            // y = sum_c head[c] (relu(acc + bias) + skip)[c] + head[CO], by a
            // tree over the channels: c and c + 8, then 4, 2 and 1 apart, the
            // first of each pair fused
            const f32x4 a = acc[m][0];
            const float4 k = skv[m][0];
            const float v[4] = {fmaxf(a[0] + bias[0].x, 0.f) + k.x, fmaxf(a[1] + bias[0].y, 0.f) + k.y,
                                fmaxf(a[2] + bias[0].z, 0.f) + k.z, fmaxf(a[3] + bias[0].w, 0.f) + k.w};
            float t[4];
#pragma unroll
            for (int e = 0; e < 4; ++e) {
              const float w = p.head[c0 + e];
              t[e] = __builtin_fmaf(v[e], w, __shfl_xor(__fmul_rn(v[e], w), 32));
              t[e] += __shfl_xor(t[e], 16);
            }
            const float h = (t[0] + t[2]) + (t[1] + t[3]);
            if (ok && kq == 0) p.y[o] = h + p.head[CO];
            continue;
          }
        }
#pragma unroll
        for (int n = 0; n < NTB; ++n) {
          const long oc = o * CO + c0 + n * 16;
          f32x4& r = acc[m][n];
          if constexpr (EPI == 1) {
            r[0] = fmaxf(r[0] + bias[n].x, 0.f);
            r[1] = fmaxf(r[1] + bias[n].y, 0.f);
            r[2] = fmaxf(r[2] + bias[n].z, 0.f);
            r[3] = fmaxf(r[3] + bias[n].w, 0.f);
            if (!ok) continue;
            const float4 k = skv[m][n];
            if (p.outA) *(float4*)(p.outA + oc) = make_float4(r[0], r[1], r[2], r[3]);
            if (p.skip) *(float4*)(p.outD + oc) = make_float4(r[0] + k.x, r[1] + k.y, r[2] + k.z, r[3] + k.w);
          } else if (ok) {
            *(float4*)(p.outA + oc) = make_float4(r[0], r[1], r[2], r[3]);
          }
        }
      }
      if constexpr (POOL) {
        // 2x2 (x, y) sums of neighbouring lanes and registers, the z pairs
        // (waves 2k, 2k+1) via LDS
        __syncthreads();
        float4* ps = (float4*)smem;   // [lz][py][px][COB / 4]
#pragma unroll
        for (int py = 0; py < 2; ++py)
#pragma unroll
          for (int n = 0; n < NTB; ++n) {
            float sum[4];
#pragma unroll
            for (int e = 0; e < 4; ++e) {
              const float lo = acc[2 * py][n][e], hi = acc[2 * py + 1][n][e];
              sum[e] = (lo + __shfl_xor(lo, 1)) + (hi + __shfl_xor(hi, 1));
            }
            if (!(i16 & 1))
              ps[((lz * 2 + py) * 8 + (i16 >> 1)) * (COB / 4) + n * 4 + kq] =
                  make_float4(sum[0], sum[1], sum[2], sum[3]);
          }
        __syncthreads();
        const int cnx = g.nx >> 1, cny = g.ny >> 1, cnz = g.nz >> 1;
        for (int q = threadIdx.x; q < 8 * COB; q += 256) {
          const int c4 = q % (COB / 4), cell = q / (COB / 4);
          const int px = cell & 7, py = (cell >> 3) & 1, pz = cell >> 4;
          const int cx = (tx0 >> 1) + px, cy = (ty >> 1) + py, cz = (tz0 >> 1) + pz;
          if (cx >= cnx || cy >= cny || cz >= cnz) continue;
          const float4 lo = ps[((2 * pz * 2 + py) * 8 + px) * (COB / 4) + c4];
          const float4 hi = ps[(((2 * pz + 1) * 2 + py) * 8 + px) * (COB / 4) + c4];
          *(float4*)(p.pool + ((long)tb * cnx * cny * cnz + cx + (long)cnx * (cy + (long)cny * cz)) * CO + nb * COB +
                     4 * c4) = make_float4(0.125f * (lo.x + hi.x), 0.125f * (lo.y + hi.y), 0.125f * (lo.z + hi.z),
                                           0.125f * (lo.w + hi.w));
        }
      }
    } else {
      // partial tiles to LDS, summed in wave order by all threads
      __syncthreads();
      float4* red = (float4*)smem;   // [wave][voxel][COB / 4]
#pragma unroll
      for (int m = 0; m < 4; ++m)
#pragma unroll
        for (int n = 0; n < NTB; ++n)
          red[((size_t)wave * 64 + m * 16 + i16) * (COB / 4) + n * 4 + kq] =
              make_float4(acc[m][n][0], acc[m][n][1], acc[m][n][2], acc[m][n][3]);
      __syncthreads();
      for (int q = threadIdx.x; q < 16 * COB; q += 256) {
        const int vox = q / (COB / 4), co = nb * COB + q % (COB / 4) * 4;
        const int vx = tx0 + (vox & 15), vy = ty + (vox >> 4);
        if (vx >= g.nx || vy >= g.ny) continue;
        const long o = ((long)tb * V + vx + (long)g.nx * (vy + (long)g.ny * tz0)) * CO + co;
        float4 r = red[q];
#pragma unroll
        for (int w = 1; w < KS; ++w) {
          const float4 t = red[(size_t)w * 16 * COB + q];
          r.x += t.x; r.y += t.y; r.z += t.z; r.w += t.w;
        }
        if (EPI == 1) {
          r.x = fmaxf(r.x + p.bias[co], 0.f);
          r.y = fmaxf(r.y + p.bias[co + 1], 0.f);
          r.z = fmaxf(r.z + p.bias[co + 2], 0.f);
          r.w = fmaxf(r.w + p.bias[co + 3], 0.f);
          if (p.outA) *(float4*)(p.outA + o) = r;
          if (p.skip) {
            const float4 k = *(const float4*)(p.skip + o);
            *(float4*)(p.outD + o) = make_float4(r.x + k.x, r.y + k.y, r.z + k.z, r.w + k.w);
          }
        } else {
          *(float4*)(p.outA + o) = r;
        }
      }
    }
  }
}

// Weight gradient: dW[t][ci][co] = sum over voxels v of X~[v + off_t][ci]
// dZ[v][co], a GEMM with K = voxels on v_mfma_f32_16x16x32_bf16 (A: row ci =
// lane % 16, B: column co = lane % 16, both k = 8 (lane / 16) + e).  A
// workgroup takes CIB input and 16 output channels and every nwg-th tile of
// 16 x 4 x 4 voxels; it stages the tile's dZ and X~ with a one-voxel halo in
// LDS as BF16, transposed to [channel][voxel] (pairs of x-neighbours packed
// as they are read), so that a lane's eight k values, eight voxels along x,
// are one 16-byte read, and each value is read from memory about 2.5 times
// instead of 27.  Its three waves take the three dz; per K-step of two rows
// a wave reads dZ once and X~ once per dy, and the dx = -1, +1 operands are
// funnel shifts of the dx = 0 one and a neighbour on either side.  The 27 /
// 3 * CIB / 16 accumulators stay in registers over all of the workgroup's
// tiles; its partial sums are added up in a fixed order by
// partial_sum_kernel.  The bias gradient sums dZ in FP32 as it is staged.
// The K loop is bound by LDS reads and MFMA issue alike (per K-step, CIB =
// 32: 80 LDS against 288 MFMA cycles a wave, three waves a workgroup on four
// SIMDs).  Four samples of 64x64x32: 50 us for 32 to 16 channels and 24 for 3
// to 16, against 530 each with one workgroup per 2,048 voxels and tap reading
// both operands from memory.
//
// LDS rows of X~: 24 values for x0 - 8 .. x0 + 15 plus the first two of the
// next row for x0 + 16, x0 + 17; 36 rows (6 y, 6 z).  Channel strides of 436
// and 132 words keep the 16-byte reads of 16 channels on distinct banks.
constexpr int WX = 436, WZ = 132;   // words per channel

struct WgradArgs {
  Geo g;
  const float* X;      // [batch][voxel][cs] (half-resolution grid when UP)
  const float* dZ;     // [batch][voxel][co]
  int cs, ci, co;      // channels of X in memory, of the gradient (padded), of dZ
  int nwg;             // workgroups per (input, output) channel block
  float* part;         // [nwg][27 * ci * co + co]
};

template <int CIB, int CSRC, bool UP>
__global__ __launch_bounds__(192) void wgrad_kernel(WgradArgs p) {
  constexpr int MB = CIB / 16, CQ = CSRC < 4 ? 1 : CIB / 4;   // channel quads staged
  __shared__ __align__(16) unsigned xs[CIB * WX];
  __shared__ __align__(16) unsigned zs[16 * WZ];
  const Geo& g = p.g;
  const int tid = threadIdx.x, wave = tid >> 6, lane = tid & 63, i16 = lane & 15, kq = lane >> 4;
  const int ncog = p.co / 16;
  const int ci0 = (blockIdx.y / ncog) * CIB, co0 = (blockIdx.y % ncog) * 16;
  const int ntx = (g.nx + 15) / 16, nty = (g.ny + 3) / 4, ntz = (g.nz + 3) / 4;
  const int ntile = ntx * nty * ntz * g.batch;
  const int sx = UP ? g.nx >> 1 : g.nx, sy = UP ? g.ny >> 1 : g.ny, sz = UP ? g.nz >> 1 : g.nz;
  if (CSRC < 4)   // channels past the source's stay zero
    for (int q = tid; q < CIB * WX; q += 192) xs[q] = 0u;
  f32x4 acc[3][3][MB];
#pragma unroll
  for (int a = 0; a < 3; ++a)
#pragma unroll
    for (int b = 0; b < 3; ++b)
#pragma unroll
      for (int m = 0; m < MB; ++m) acc[a][b][m] = f32x4{0.f, 0.f, 0.f, 0.f};
  float4 bsum = make_float4(0.f, 0.f, 0.f, 0.f);   // this thread's channel quad of dZ
  for (int tile = blockIdx.x; tile < ntile; tile += p.nwg) {
    const int tx = tile % ntx, ty = (tile / ntx) % nty, tz = (tile / (ntx * nty)) % ntz, b = tile / (ntx * nty * ntz);
    const int x0 = tx * 16, y0 = ty * 4, z0 = tz * 4;
    const float* Xb = p.X + (long)b * sx * sy * sz * p.cs + ci0;
    const float* Zb = p.dZ + (long)b * g.V * p.co + co0;
    __syncthreads();   // the previous tile's reads are done
    constexpr int NX = 36 * 10 * CQ, U = 5;
    for (int q0 = 0; q0 < NX; q0 += U * 192) {
      float4 lo[U], hi[U];
#pragma unroll
      for (int u = 0; u < U; ++u) {
        const int q = q0 + u * 192 + tid;
        lo[u] = hi[u] = make_float4(0.f, 0.f, 0.f, 0.f);
        if (q >= NX) continue;
        const int c4 = (q % CQ) * 4, pr = q / CQ, row = pr / 10;
        const int x = x0 + 2 * (pr % 10) - 2, y = y0 + row % 6 - 1, z = z0 + row / 6 - 1;
        if (y < 0 || y >= g.ny || z < 0 || z >= g.nz) continue;
        auto load = [&](int xx) {
          const float* src =
              UP ? Xb + ((long)(xx >> 1) + (long)sx * ((y >> 1) + (long)sy * (z >> 1))) * p.cs + c4
                 : Xb + ((long)xx + (long)sx * (y + (long)sy * z)) * p.cs + c4;
          if (CSRC < 4) return make_float4(src[0], src[1], src[2], 0.f);
          return *(const float4*)src;
        };
        if (x >= 0 && x < g.nx) lo[u] = load(x);
        if (x + 1 >= 0 && x + 1 < g.nx) hi[u] = UP ? lo[u] : load(x + 1);   // x is even
      }
#pragma unroll
      for (int u = 0; u < U; ++u) {
        const int q = q0 + u * 192 + tid;
        if (q >= NX) continue;
        const int c4 = (q % CQ) * 4, pr = q / CQ;
        unsigned* d = xs + c4 * WX + (pr / 10) * 12 + pr % 10 + 3;
        d[0] = pack_bf16x2(lo[u].x, hi[u].x);
        d[WX] = pack_bf16x2(lo[u].y, hi[u].y);
        d[2 * WX] = pack_bf16x2(lo[u].z, hi[u].z);
        if (CSRC >= 4) d[3 * WX] = pack_bf16x2(lo[u].w, hi[u].w);
      }
    }
#pragma unroll
    for (int u = 0; u < 3; ++u) {   // 16 rows of 8 pairs, 4 channel quads
      const int q = u * 192 + tid;
      if (q >= 512) continue;
      const int c4 = (q & 3) * 4, pr = q >> 2, row = pr >> 3;
      const int x = x0 + 2 * (pr & 7), y = y0 + (row & 3), z = z0 + (row >> 2);
      float4 lo = make_float4(0.f, 0.f, 0.f, 0.f), hi = lo;
      if (y < g.ny && z < g.nz) {
        const float* src = Zb + ((long)x + (long)g.nx * (y + (long)g.ny * z)) * p.co + c4;
        if (x < g.nx) lo = *(const float4*)src;
        if (x + 1 < g.nx) hi = *(const float4*)(src + p.co);
      }
      bsum.x += lo.x + hi.x;
      bsum.y += lo.y + hi.y;
      bsum.z += lo.z + hi.z;
      bsum.w += lo.w + hi.w;
      unsigned* d = zs + c4 * WZ + row * 8 + (pr & 7);
      d[0] = pack_bf16x2(lo.x, hi.x);
      d[WZ] = pack_bf16x2(lo.y, hi.y);
      d[2 * WZ] = pack_bf16x2(lo.z, hi.z);
      d[3 * WZ] = pack_bf16x2(lo.w, hi.w);
    }
    __syncthreads();
#pragma unroll 2
    for (int ks = 0; ks < 8; ++ks) {
      const int z = ks >> 1, y = (ks & 1) * 2 + (kq >> 1), xh = kq & 1;
      const bf16x8 bz = __builtin_bit_cast(bf16x8, *(const uint4*)(zs + i16 * WZ + (z * 4 + y) * 8 + xh * 4));
#pragma unroll
      for (int dy = 0; dy < 3; ++dy)
#pragma unroll
        for (int m = 0; m < MB; ++m) {
          const unsigned* r = xs + (m * 16 + i16) * WX + ((z + wave) * 6 + y + dy) * 12 + 4 + xh * 4;
          const uint4 c = *(const uint4*)r;
          const unsigned l = r[-1], t = r[4];
          const unsigned s1 = __builtin_amdgcn_alignbit(c.y, c.x, 16), s2 = __builtin_amdgcn_alignbit(c.z, c.y, 16),
                         s3 = __builtin_amdgcn_alignbit(c.w, c.z, 16);
          const uint4 am = make_uint4(__builtin_amdgcn_alignbit(c.x, l, 16), s1, s2, s3);
          const uint4 ap = make_uint4(s1, s2, s3, __builtin_amdgcn_alignbit(t, c.w, 16));
          acc[dy][0][m] = __builtin_amdgcn_mfma_f32_16x16x32_bf16(__builtin_bit_cast(bf16x8, am), bz, acc[dy][0][m], 0, 0, 0);
          acc[dy][1][m] = __builtin_amdgcn_mfma_f32_16x16x32_bf16(__builtin_bit_cast(bf16x8, c), bz, acc[dy][1][m], 0, 0, 0);
          acc[dy][2][m] = __builtin_amdgcn_mfma_f32_16x16x32_bf16(__builtin_bit_cast(bf16x8, ap), bz, acc[dy][2][m], 0, 0, 0);
        }
    }
  }
  // C element (row 4 * kq + e, column i16): input channel, output channel
  const size_t per = (size_t)27 * p.ci * p.co;
  float* out = p.part + (size_t)blockIdx.x * (per + p.co);
#pragma unroll
  for (int dy = 0; dy < 3; ++dy)
#pragma unroll
    for (int dx = 0; dx < 3; ++dx)
#pragma unroll
      for (int m = 0; m < MB; ++m)
#pragma unroll
        for (int e = 0; e < 4; ++e)
          out[((size_t)(wave * 9 + dy * 3 + dx) * p.ci + ci0 + m * 16 + 4 * kq + e) * p.co + co0 + i16] =
              acc[dy][dx][m][e];
  if (ci0 == 0) {
    __syncthreads();
    float* sh = (float*)zs;   // [48][16]
    *(float4*)(sh + 4 * tid) = bsum;
    __syncthreads();
    if (tid < 16) {
      float t = 0.f;
      for (int q = 0; q < 48; ++q) t += sh[q * 16 + tid];
      out[per + co0 + tid] = t;
    }
  }
}

// The gradient of one convolution's parameters (weights of its real input
// channels, then biases), or any rows of `width` partial sums: out[q] = sum
// over the n partials of column src(q), 32 columns a block, eight rows of
// threads taking every eighth partial; fixed order.
__global__ __launch_bounds__(256) void partial_sum_kernel(int n, size_t width, const float* __restrict__ part,
                                                          int nout, int ci_pad, int ci_real, int co,
                                                          float* __restrict__ out) {
  __shared__ float sh[8][32];
  const int lane = threadIdx.x & 31, row = threadIdx.x >> 5;
  const int q = blockIdx.x * 32 + lane;
  float s = 0.f;
  if (q < nout) {
    size_t src = q;
    if (ci_pad) {   // out [27][ci_real][co], co; part [27][ci_pad][co], co
      const int per = ci_real * co, t = q / per;
      src = t < 27 ? (size_t)t * ci_pad * co + q % per : (size_t)27 * ci_pad * co + (q - 27 * per);
    }
#pragma unroll 8
    for (int k = row; k < n; k += 8) s += part[(size_t)k * width + src];
  }
  sh[row][lane] = s;
  __syncthreads();
  if (row == 0 && q < nout) {
    float t = 0.f;
#pragma unroll
    for (int r = 0; r < 8; ++r) t += sh[r][lane];
    out[q] = t;
  }
}

// ------------------------------------------------------------ elementwise
// 2x2x2 average pooling of X on grid g2 = 2 * (output grid g).
__global__ void pool_kernel(Geo g, int C, const float* __restrict__ X, float* __restrict__ out) {
  long q = (long)blockIdx.x * blockDim.x + threadIdx.x;
  long total = (long)g.batch * g.V * C;
  if (q >= total) return;
  int c = (int)(q % C);
  long bv = q / C;
  int b = (int)(bv / g.V), v = (int)(bv % g.V);
  int x = v % g.nx, yz = v / g.nx, y = yz % g.ny, z = yz / g.ny;
  int fx = 2 * g.nx, fy = 2 * g.ny, fV = 8 * g.V;
  float s = 0.f;
  for (int k = 0; k < 2; ++k)
    for (int j = 0; j < 2; ++j)
      for (int i = 0; i < 2; ++i)
        s += X[((long)b * fV + (2 * x + i) + (long)fx * ((2 * y + j) + (long)fy * (2 * z + k))) * C + c];
  out[q] = s * 0.125f;
}

// The backward elementwise passes take four channels a thread and write the
// gradient behind the ReLU, dZ = G (a > 0), as they form G, so that no pass
// reads G back only to mask it.
__device__ inline float4 relu_mask(float4 g, float4 a) {
  return make_float4(a.x > 0.f ? g.x : 0.f, a.y > 0.f ? g.y : 0.f, a.z > 0.f ? g.z : 0.f, a.w > 0.f ? g.w : 0.f);
}

// Encoder gradient G = dX + (coarse gradient of the pooled tensor) / 8,
// masked by the activation a.  dX given, or (level 0) dy wo of the head.
template <int C, bool HEAD>
__global__ __launch_bounds__(256) void pool_bwd_kernel(Geo fine, const float* __restrict__ dP,
                                                       const float* __restrict__ dX, const float* __restrict__ wb,
                                                       const float* __restrict__ a, float* __restrict__ dZ) {
  const long q = (long)blockIdx.x * blockDim.x + threadIdx.x;
  if (q >= (long)fine.batch * fine.V * (C / 4)) return;
  const int c4 = (int)(q % (C / 4)) * 4;
  const long bv = q / (C / 4);
  const int b = (int)(bv / fine.V), v = (int)(bv - (long)b * fine.V);
  const int x = v % fine.nx, yz = v / fine.nx, y = yz % fine.ny, z = yz / fine.ny;
  const int cnx = fine.nx / 2, cny = fine.ny / 2, cV = fine.V / 8;
  const float4 d =
      *(const float4*)(dP + ((long)b * cV + (x >> 1) + (long)cnx * ((y >> 1) + (long)cny * (z >> 1))) * C + c4);
  float4 g;
  if (HEAD) {
    const float h = dX[bv];
    g = make_float4(h * wb[c4], h * wb[c4 + 1], h * wb[c4 + 2], h * wb[c4 + 3]);
  } else {
    g = *(const float4*)(dX + bv * C + c4);
  }
  g.x += d.x * 0.125f;
  g.y += d.y * 0.125f;
  g.z += d.z * 0.125f;
  g.w += d.w * 0.125f;
  *(float4*)(dZ + bv * C + c4) = relu_mask(g, *(const float4*)(a + bv * C + c4));
}

// Coarse gradient G of an upsampled tensor: sum of its 8 children (g
// coarse), stored in out when given and masked by a in dZ.
template <int C>
__global__ __launch_bounds__(256) void up_bwd_kernel(Geo g, const float* __restrict__ dU, const float* __restrict__ a,
                                                     float* __restrict__ out, float* __restrict__ dZ) {
  const long q = (long)blockIdx.x * blockDim.x + threadIdx.x;
  if (q >= (long)g.batch * g.V * (C / 4)) return;
  const int c4 = (int)(q % (C / 4)) * 4;
  const long bv = q / (C / 4);
  const int b = (int)(bv / g.V), v = (int)(bv - (long)b * g.V);
  const int x = v % g.nx, yz = v / g.nx, y = yz % g.ny, z = yz / g.ny;
  const int fx = 2 * g.nx, fy = 2 * g.ny, fV = 8 * g.V;
  float4 s = make_float4(0.f, 0.f, 0.f, 0.f);
#pragma unroll
  for (int e = 0; e < 8; ++e) {
    const float4 d = *(const float4*)(
        dU + ((long)b * fV + (2 * x + (e & 1)) + (long)fx * ((2 * y + ((e >> 1) & 1)) + (long)fy * (2 * z + (e >> 2)))) * C + c4);
    s.x += d.x;
    s.y += d.y;
    s.z += d.z;
    s.w += d.w;
  }
  if (out) *(float4*)(out + bv * C + c4) = s;
  *(float4*)(dZ + bv * C + c4) = relu_mask(s, *(const float4*)(a + bv * C + c4));
}

// Head: y[v] = sum_c d0[v][c] wo[c] + bo.
__global__ void head_fwd_kernel(long nvox, const float* __restrict__ d0, const float* __restrict__ wb,
                                float* __restrict__ y) {
  long v = (long)blockIdx.x * blockDim.x + threadIdx.x;
  if (v >= nvox) return;
  float s = 0.f;
#pragma unroll
  for (int c = 0; c < 16; ++c) s += d0[v * 16 + c] * wb[c];
  y[v] = s + wb[16];
}

// Head backward: dZ[v][c] = dy[v] wo[c] (a6 > 0), and per block the partial
// sums of the head's own gradient, d0[v][c] dy[v] and dy[v].
constexpr int HEAD_BLOCKS = 512;
__global__ __launch_bounds__(256) void head_bwd_kernel(long nvox, const float* __restrict__ d0,
                                                       const float* __restrict__ dy, const float* __restrict__ wb,
                                                       const float* __restrict__ a6, float* __restrict__ dZ,
                                                       float* __restrict__ part) {
  __shared__ float sh[256][5];
  const int c4 = (threadIdx.x & 3) * 4;
  const float4 w = make_float4(wb[c4], wb[c4 + 1], wb[c4 + 2], wb[c4 + 3]);
  float4 s = make_float4(0.f, 0.f, 0.f, 0.f);
  float sy = 0.f;
  for (long v = (long)blockIdx.x * 64 + (threadIdx.x >> 2); v < nvox; v += (long)gridDim.x * 64) {
    const float h = dy[v];
    const float4 d = *(const float4*)(d0 + v * 16 + c4);
    *(float4*)(dZ + v * 16 + c4) =
        relu_mask(make_float4(h * w.x, h * w.y, h * w.z, h * w.w), *(const float4*)(a6 + v * 16 + c4));
    s.x += d.x * h;
    s.y += d.y * h;
    s.z += d.z * h;
    s.w += d.w * h;
    sy += h;
  }
  float* r = sh[threadIdx.x];
  r[0] = s.x; r[1] = s.y; r[2] = s.z; r[3] = s.w; r[4] = sy;
  __syncthreads();
  if (threadIdx.x < 17) {
    const int c = threadIdx.x;
    float t = 0.f;
    for (int q = 0; q < 64; ++q) t += c < 16 ? sh[4 * q + (c >> 2)][c & 3] : sh[4 * q][4];
    part[(size_t)blockIdx.x * 17 + c] = t;
  }
}

// Loss partials per sample over a block's voxels: y.t, y.y, t.t.
__global__ void loss_partial_kernel(int V, int nblk_per, const float* __restrict__ y, const float* __restrict__ t,
                                    float* __restrict__ part) {
  __shared__ float s1[256], s2[256], s3[256];
  int b = blockIdx.x / nblk_per, k = blockIdx.x % nblk_per;
  long per = (V + nblk_per - 1) / nblk_per;
  long beg = (long)k * per, end = beg + per < V ? beg + per : V;
  float a = 0.f, c = 0.f, e = 0.f;
  for (long v = beg + threadIdx.x; v < end; v += 256) {
    float yv = y[(long)b * V + v], tv = t[(long)b * V + v];
    a += yv * tv;
    c += yv * yv;
    e += tv * tv;
  }
  s1[threadIdx.x] = a;
  s2[threadIdx.x] = c;
  s3[threadIdx.x] = e;
  __syncthreads();
  for (int o = 128; o > 0; o >>= 1) {
    if (threadIdx.x < o) {
      s1[threadIdx.x] += s1[threadIdx.x + o];
      s2[threadIdx.x] += s2[threadIdx.x + o];
      s3[threadIdx.x] += s3[threadIdx.x + o];
    }
    __syncthreads();
  }
  if (threadIdx.x == 0) {
    part[3 * blockIdx.x] = s1[0];
    part[3 * blockIdx.x + 1] = s2[0];
    part[3 * blockIdx.x + 2] = s3[0];
  }
}

// Per-sample totals (fixed order); the direction loss
// L = mean_b (1 - (y.t)^2 / (|y|^2 |t|^2)) and
// dy = -(2/B) [c t - c (y.t)/|y|^2 y], c = (y.t) / (|y|^2 |t|^2).
__global__ void loss_grad_kernel(int B, int V, int nblk_per, const float* __restrict__ part,
                                 const float* __restrict__ y, const float* __restrict__ t, float* __restrict__ dy,
                                 float* __restrict__ loss) {
  __shared__ float yt[64], yy[64], tt[64];
  if (threadIdx.x < B) {
    float a = 0.f, c = 0.f, e = 0.f;
    for (int k = 0; k < nblk_per; ++k) {
      a += part[3 * (threadIdx.x * nblk_per + k)];
      c += part[3 * (threadIdx.x * nblk_per + k) + 1];
      e += part[3 * (threadIdx.x * nblk_per + k) + 2];
    }
    yt[threadIdx.x] = a;
    yy[threadIdx.x] = c;
    tt[threadIdx.x] = e;
  }
  __syncthreads();
  if (blockIdx.x == 0 && threadIdx.x == 0) {
    float L = 0.f;
    for (int b = 0; b < B; ++b) L += 1.f - yt[b] * yt[b] / (yy[b] * tt[b]);
    *loss = L / B;
  }
  for (long q = (long)blockIdx.x * blockDim.x + threadIdx.x; q < (long)B * V; q += (long)gridDim.x * blockDim.x) {
    int b = (int)(q / V);
    float c = yt[b] / (yy[b] * tt[b]);
    dy[q] = -(2.f / B) * (c * t[q] - (c * yt[b] / yy[b]) * y[q]);
  }
}

// Training target: t = e / s in FP32.
__global__ void target_kernel(long n, const double* __restrict__ e, double inv, float* __restrict__ t) {
  long q = (long)blockIdx.x * blockDim.x + threadIdx.x;
  if (q < n) t[q] = (float)(e[q] * inv);
}

// Adam with bias correction; c1 = 1/(1 - b1^k), c2 = 1/(1 - b2^k).
__global__ void adam_kernel(long n, float lr, float b1, float b2, float eps, float c1, float c2,
                            const float* __restrict__ g, float* __restrict__ m, float* __restrict__ v,
                            float* __restrict__ w) {
  long q = (long)blockIdx.x * blockDim.x + threadIdx.x;
  if (q >= n) return;
  float gq = g[q];
  float mq = b1 * m[q] + (1.f - b1) * gq;
  float vq = b2 * v[q] + (1.f - b2) * gq * gq;
  m[q] = mq;
  v[q] = vq;
  w[q] -= lr * (mq * c1) / (sqrtf(vq * c2) + eps);
}

// (tap, channel) of K-index kk (0..31) of K-step ks for a convolution whose
// K side has ck channels (the ordering the convolution kernel reads).
__device__ inline void k_index(int ck, int ks, int kk, int& t, int& c) {
  if (ck >= 32) {
    t = ks / (ck / 32);
    c = (ks % (ck / 32)) * 32 + kk;
  } else if (ck == 16) {
    t = 2 * ks + (kk >> 4);
    c = kk & 15;
  } else {
    const int k = ks * 32 + kk;
    t = k >> 2;
    c = k & 3;
  }
}

// BF16 fragments of conv weights W[27][ci][co] (FP32 master) for
// v_mfma_f32_16x16x32_bf16: frag[ks][nt][lane][e] is the weight at K-index
// kk = 8*(lane/16) + e of step ks and result channel nt*16 + lane%16.
// Forward: K = (tap, ci) with ck = 4 for the 3-channel input, M = co.
// Backward (data gradient): taps mirrored (26 - t), K = (tap, co), M = ci.
__global__ void frag_kernel(int ci, int ck, int co, int backward, const float* __restrict__ W,
                            bf16x8* __restrict__ frag) {
  const int nt_n = backward ? ci / 16 : co / 16;
  const int kside = backward ? co : ck;
  const int q = blockIdx.x * blockDim.x + threadIdx.x;
  if (q >= ksteps(kside) * nt_n * 64) return;
  const int lane = q % 64, nt = (q / 64) % nt_n, ks = q / (64 * nt_n);
  const int n = nt * 16 + lane % 16;
  bf16x8 f;
  for (int e = 0; e < 8; ++e) {
    int t, c;
    k_index(kside, ks, 8 * (lane / 16) + e, t, c);
    float w = 0.f;
    if (t < 27) {
      if (!backward && c < ci) w = W[((size_t)t * ci + c) * co + n];
      if (backward) w = W[((size_t)(26 - t) * ci + n) * co + c];
    }
    f[e] = __builtin_bit_cast(__bf16, (unsigned short)f2bf(w));
  }
  frag[q] = f;
}

}  // namespace

// ------------------------------------------------------------ host object

struct cpr_nn {
  std::string err;
  DevAlloc mem;        // device allocator taken at creation
  hipStream_t stream = nullptr;
  Geo lv[4];           // grid per level (batch = max_batch)
  int max_batch = 0;
  long P = 0;
  long off[NCONV + 1]; // parameter offsets: conv k weights at off[k], bias after
  float* theta = nullptr;
  float* m = nullptr;
  float* vv = nullptr;
  float* grad = nullptr;
  bf16x8* wf[NCONV] = {};
  bf16x8* wb[NCONV] = {};
  // activations
  float *x3 = nullptr, *e0 = nullptr, *p1 = nullptr, *e1 = nullptr, *p2 = nullptr, *e2 = nullptr;
  float *p3 = nullptr, *e3 = nullptr, *a4 = nullptr, *d2 = nullptr, *a5 = nullptr, *d1 = nullptr;
  float *a6 = nullptr, *d0 = nullptr, *y = nullptr;
  // gradients
  float *dy = nullptr, *g0b = nullptr, *gu0 = nullptr, *g1 = nullptr, *g1b = nullptr;
  float *gu1 = nullptr, *g2 = nullptr, *g2b = nullptr, *gu2 = nullptr, *g3b = nullptr;
  float *part = nullptr, *lpart = nullptr, *loss = nullptr;
  size_t part_cap = 0;
  int cur_batch = 0;
  long adam_step = 0;
  bool frags_valid = false;
};

static int nn_err(cpr_nn* nn, int code, const std::string& msg) {
  if (nn) nn->err = msg;
  return code;
}

#define NN_TRY(expr)                                                            \
  do {                                                                          \
    hipError_t e_ = (expr);                                                     \
    if (e_ != hipSuccess) return nn_err(nn, CPR_EHIP, std::string(#expr) + ": " + hipGetErrorString(e_)); \
  } while (0)

static long nn_param_count() {
  long p = 0;
  for (int k = 0; k < NCONV; ++k) p += 27L * CIN[k] * COUT[k] + COUT[k];
  return p + 17;
}

static Geo with_batch(Geo g, int b) { g.batch = b; return g; }

static int fwd_frags(int k) { return ksteps(k == 0 ? 4 : CIN[k]) * (COUT[k] / 16) * 64; }
static int bwd_frags(int k) { return ksteps(COUT[k]) * (CIN[k] / 16) * 64; }

static int nn_refresh_frags(cpr_nn* nn) {
  for (int k = 0; k < NCONV; ++k) {
    const float* W = nn->theta + nn->off[k];
    frag_kernel<<<div_up(fwd_frags(k), 256), 256, 0, nn->stream>>>(CIN[k], k == 0 ? 4 : CIN[k], COUT[k], 0, W,
                                                                   nn->wf[k]);
    if (k > 0)
      frag_kernel<<<div_up(bwd_frags(k), 256), 256, 0, nn->stream>>>(CIN[k], CIN[k], COUT[k], 1, W, nn->wb[k]);
  }
  nn->frags_valid = true;
  NN_TRY(hipGetLastError());
  return CPR_OK;
}

// Grids of at least 64K voxels use whole-tile waves (K split 1); smaller
// ones, and 64-channel inputs at full resolution (whose LDS window would
// not fit beside the weights), split the K-steps over the 4 waves of a
// workgroup.  The output channels are split over NS workgroups so that a
// workgroup's weight fragments fit in 56 KB of LDS and, where the channels
// allow, the launch has at least 512 workgroups.
constexpr int WMAX = 56 * 1024;
constexpr int wbytes(int ci, int co, int ns) { return ksteps(ci) * (co / (16 * ns)) * 1024; }

static ConvArgs cargs(Geo g, const float* X, const bf16x8* W, const float* bias, const float* skip, float* outA,
                      float* outD) {
  ConvArgs a{};
  a.g = g; a.X = X; a.W = W; a.bias = bias; a.skip = skip; a.outA = outA; a.outD = outD;
  return a;
}

// With KS = 1 a workgroup walks over its share of the tiles, and there are as
// many as the chip holds (KS = 4: one per tile).
template <int CI, int CSRC, int CO, bool UP, int EPI, int KS, int NS, bool POOL>
static void conv_launch(cpr_nn* nn, const ConvArgs& a, long tiles) {
  constexpr long resident = (long)CUS * conv_per_cu<CI, CO, UP, KS, NS>() / NS;
  const long walkers = KS == 1 ? std::min(tiles, resident) : tiles;
  conv_kernel<CI, CSRC, CO, UP, EPI, KS, NS, POOL><<<walkers * NS, 256, 0, nn->stream>>>(a);
}

template <int CI, int CSRC, int CO, bool UP, int EPI, int KS, bool POOL>
static void conv_ns(cpr_nn* nn, const ConvArgs& a, long tiles, int ns) {
  if constexpr (wbytes(CI, CO, 1) <= WMAX)
    if (ns == 1) {
      conv_launch<CI, CSRC, CO, UP, EPI, KS, 1, POOL>(nn, a, tiles);
      return;
    }
  if constexpr (CO >= 32 && wbytes(CI, CO, 2) <= WMAX)
    if (ns == 2) {
      conv_launch<CI, CSRC, CO, UP, EPI, KS, 2, POOL>(nn, a, tiles);
      return;
    }
  if constexpr (CO >= 64)
    if (ns == 4) conv_launch<CI, CSRC, CO, UP, EPI, KS, 4, POOL>(nn, a, tiles);
}

// a.pool (POOL only): also write the 2x2x2 average of the activations,
// fused when the tiles hold whole cells, else by a separate pass.
template <int CI, int CSRC, int CO, bool UP, int EPI, bool POOL = false>
static void conv(cpr_nn* nn, ConvArgs a) {
  const Geo& g = a.g;
  const long vox = (long)g.batch * g.V;
  const long txy = (long)div_up(g.nx, TX) * div_up(g.ny, TY);
  constexpr bool fits = UP || CI <= 32;
  const bool whole = fits && vox >= 65536;
  const long tiles = whole ? txy * div_up(g.nz, 4) * g.batch : txy * g.nz * g.batch;
  int ns = 1;
  while (wbytes(CI, CO, ns) > WMAX) ns *= 2;
  while (CO / (16 * ns) >= 2 && ns < 4 && tiles * ns < 512) ns *= 2;
  if constexpr (fits)
    if (whole) {
      conv_ns<CI, CSRC, CO, UP, EPI, 1, POOL>(nn, a, tiles, ns);
      return;
    }
  ConvArgs b = a;
  b.head = nullptr;
  b.y = nullptr;
  b.pool = nullptr;
  conv_ns<CI, CSRC, CO, UP, EPI, 4, false>(nn, b, tiles, ns);
  if (POOL) {
    Geo c = g;
    c.nx >>= 1; c.ny >>= 1; c.nz >>= 1;
    c.V = c.nx * c.ny * c.nz;
    pool_kernel<<<div_up((long)g.batch * c.V * CO, 256), 256, 0, nn->stream>>>(c, CO, a.outA, a.pool);
  }
}

// Workgroups per channel block of a weight gradient: at most one per tile,
// WG_MAX over all blocks (two per CU: 64 KB of LDS each; more would only add
// partial sums, 55 KB apiece, to the reduction).
static int wgrad_wgs(const Geo& g, int ci_pad, int co) {
  const int cib = ci_pad < 32 ? ci_pad : 32, blocks = (ci_pad / cib) * (co / 16);
  const int tiles = div_up(g.nx, 16) * div_up(g.ny, 4) * div_up(g.nz, 4) * g.batch;
  return std::min(tiles, WG_MAX / blocks);
}

// Gradient of convolution k's parameters from its input X and dZ.
template <int CI, int CSRC, int CO, bool UP>
static void wgrad(cpr_nn* nn, Geo g, const float* X, const float* dZ, int k) {
  constexpr int CIB = CI < 32 ? CI : 32;
  WgradArgs a;
  a.g = g; a.X = X; a.dZ = dZ;
  a.cs = CSRC; a.ci = CI; a.co = CO;
  a.nwg = wgrad_wgs(g, CI, CO);
  a.part = nn->part;
  wgrad_kernel<CIB, CSRC, UP><<<dim3(a.nwg, (CI / CIB) * (CO / 16)), 192, 0, nn->stream>>>(a);
  const int nout = 27 * CSRC * CO + CO;
  partial_sum_kernel<<<div_up(nout, 32), 256, 0, nn->stream>>>(a.nwg, (size_t)27 * CI * CO + CO, nn->part, nout, CI,
                                                             CSRC, CO, nn->grad + nn->off[k]);
}

// x3: input features [B][voxel][3].  train: keep what the backward pass
// needs (pre-skip activations, d0) and run the head separately; otherwise
// only what inference needs, with the head fused into the last convolution.
static int nn_forward_impl(cpr_nn* nn, const float* x3, int B, bool train, const double* xscale = nullptr) {
  Geo L0 = with_batch(nn->lv[0], B), L1 = with_batch(nn->lv[1], B), L2 = with_batch(nn->lv[2], B),
      L3 = with_batch(nn->lv[3], B);
  hipStream_t s = nn->stream;
  auto bias = [&](int k) { return nn->theta + nn->off[k] + 27L * CIN[k] * COUT[k]; };
  const float* head = nn->theta + nn->off[NCONV];
  ConvArgs a = cargs(L0, x3, nn->wf[0], bias(0), nullptr, nn->e0, nullptr);
  a.pool = nn->p1;
  a.xscale = xscale;
  conv<4, 3, 16, false, 1, true>(nn, a);
  a = cargs(L1, nn->p1, nn->wf[1], bias(1), nullptr, nn->e1, nullptr);
  a.pool = nn->p2;
  conv<16, 16, 32, false, 1, true>(nn, a);
  a = cargs(L2, nn->p2, nn->wf[2], bias(2), nullptr, nn->e2, nullptr);
  a.pool = nn->p3;
  conv<32, 32, 64, false, 1, true>(nn, a);
  conv<64, 64, 64, false, 1>(nn, cargs(L3, nn->p3, nn->wf[3], bias(3), nullptr, nn->e3, nullptr));
  conv<64, 64, 64, true, 1>(nn, cargs(L2, nn->e3, nn->wf[4], bias(4), nn->e2, train ? nn->a4 : nullptr, nn->d2));
  conv<64, 64, 32, true, 1>(nn, cargs(L1, nn->d2, nn->wf[5], bias(5), nn->e1, train ? nn->a5 : nullptr, nn->d1));
  const long n0 = (long)B * L0.V;
  if (train || n0 < 65536) {
    conv<32, 32, 16, true, 1>(nn, cargs(L0, nn->d1, nn->wf[6], bias(6), nn->e0, nn->a6, nn->d0));
    head_fwd_kernel<<<div_up(n0, 256), 256, 0, s>>>(n0, nn->d0, head, nn->y);
  } else {
    a = cargs(L0, nn->d1, nn->wf[6], bias(6), nn->e0, nullptr, nullptr);
    a.head = head;
    a.y = nn->y;
    conv<32, 32, 16, true, 1>(nn, a);
  }
  nn->cur_batch = train ? B : 0;
  NN_TRY(hipGetLastError());
  return CPR_OK;
}

// Gradient of sum(dy * y) for the last forward pass into nn->grad.
static int nn_backward_impl(cpr_nn* nn) {
  const int B = nn->cur_batch;
  Geo L0 = with_batch(nn->lv[0], B), L1 = with_batch(nn->lv[1], B), L2 = with_batch(nn->lv[2], B),
      L3 = with_batch(nn->lv[3], B);
  hipStream_t s = nn->stream;
  long n0 = (long)B * L0.V, n1 = (long)B * L1.V, n2 = (long)B * L2.V, n3 = (long)B * L3.V;
  const float* head = nn->theta + nn->off[NCONV];
  auto quads = [](long nvox, int c) { return div_up(nvox * (c / 4), 256); };
  // head and level 0 decoder: d0 = a6 + e0, so dd0 = dy wo reaches a6 and e0
  const int hb = (int)std::min<long>(HEAD_BLOCKS, div_up(n0, 64));
  head_bwd_kernel<<<hb, 256, 0, s>>>(n0, nn->d0, nn->dy, head, nn->a6, nn->g0b, nn->part);
  partial_sum_kernel<<<1, 256, 0, s>>>(hb, 17, nn->part, 17, 0, 0, 0, nn->grad + nn->off[NCONV]);
  wgrad<32, 32, 16, true>(nn, L0, nn->d1, nn->g0b, 6);
  conv<16, 16, 32, false, 0>(nn, cargs(L0, nn->g0b, nn->wb[6], nullptr, nullptr, nn->gu0, nullptr));
  up_bwd_kernel<32><<<quads(n1, 32), 256, 0, s>>>(L1, nn->gu0, nn->a5, nn->g1, nn->g1b);      // dd1 = de1
  wgrad<64, 64, 32, true>(nn, L1, nn->d2, nn->g1b, 5);
  conv<32, 32, 64, false, 0>(nn, cargs(L1, nn->g1b, nn->wb[5], nullptr, nullptr, nn->gu1, nullptr));
  up_bwd_kernel<64><<<quads(n2, 64), 256, 0, s>>>(L2, nn->gu1, nn->a4, nn->g2, nn->g2b);      // dd2 = de2
  wgrad<64, 64, 64, true>(nn, L2, nn->e3, nn->g2b, 4);
  conv<64, 64, 64, false, 0>(nn, cargs(L2, nn->g2b, nn->wb[4], nullptr, nullptr, nn->gu2, nullptr));
  // encoder: de3, then de2, de1, de0 with the pooled tensors' gradients
  up_bwd_kernel<64><<<quads(n3, 64), 256, 0, s>>>(L3, nn->gu2, nn->e3, nullptr, nn->g3b);
  wgrad<64, 64, 64, false>(nn, L3, nn->p3, nn->g3b, 3);
  conv<64, 64, 64, false, 0>(nn, cargs(L3, nn->g3b, nn->wb[3], nullptr, nullptr, nn->gu2, nullptr));  // dp3 (L3)
  pool_bwd_kernel<64, false><<<quads(n2, 64), 256, 0, s>>>(L2, nn->gu2, nn->g2, nullptr, nn->e2, nn->g2b);
  wgrad<32, 32, 64, false>(nn, L2, nn->p2, nn->g2b, 2);
  conv<64, 64, 32, false, 0>(nn, cargs(L2, nn->g2b, nn->wb[2], nullptr, nullptr, nn->gu1, nullptr));  // dp2 (L2, 32)
  pool_bwd_kernel<32, false><<<quads(n1, 32), 256, 0, s>>>(L1, nn->gu1, nn->g1, nullptr, nn->e1, nn->g1b);
  wgrad<16, 16, 32, false>(nn, L1, nn->p1, nn->g1b, 1);
  conv<32, 32, 16, false, 0>(nn, cargs(L1, nn->g1b, nn->wb[1], nullptr, nullptr, nn->gu0, nullptr));  // dp1 (L1, 16)
  pool_bwd_kernel<16, true><<<quads(n0, 16), 256, 0, s>>>(L0, nn->gu0, nn->dy, head, nn->e0, nn->g0b);
  wgrad<16, 3, 16, false>(nn, L0, nn->x3, nn->g0b, 0);
  NN_TRY(hipGetLastError());
  return CPR_OK;
}

static int nn_alloc(cpr_nn* nn) {
  const int B = nn->max_batch;
  long n[4];
  for (int l = 0; l < 4; ++l) n[l] = (long)B * nn->lv[l].V;
  auto A = [&](float** p, long cnt) -> hipError_t {
    return dev_malloc(nn->mem, (void**)p, (cnt > 0 ? cnt : 1) * sizeof(float));
  };
  NN_TRY(A(&nn->theta, nn->P)); NN_TRY(A(&nn->m, nn->P)); NN_TRY(A(&nn->vv, nn->P)); NN_TRY(A(&nn->grad, nn->P));
  for (int k = 0; k < NCONV; ++k) {
    NN_TRY(dev_malloc(nn->mem, (void**)&nn->wf[k], fwd_frags(k) * sizeof(bf16x8)));
    NN_TRY(dev_malloc(nn->mem, (void**)&nn->wb[k], bwd_frags(k) * sizeof(bf16x8)));
  }
  NN_TRY(A(&nn->x3, n[0] * 3)); NN_TRY(A(&nn->e0, n[0] * 16)); NN_TRY(A(&nn->p1, n[1] * 16));
  NN_TRY(A(&nn->e1, n[1] * 32)); NN_TRY(A(&nn->p2, n[2] * 32)); NN_TRY(A(&nn->e2, n[2] * 64));
  NN_TRY(A(&nn->p3, n[3] * 64)); NN_TRY(A(&nn->e3, n[3] * 64)); NN_TRY(A(&nn->a4, n[2] * 64));
  NN_TRY(A(&nn->d2, n[2] * 64)); NN_TRY(A(&nn->a5, n[1] * 32)); NN_TRY(A(&nn->d1, n[1] * 32));
  NN_TRY(A(&nn->a6, n[0] * 16)); NN_TRY(A(&nn->d0, n[0] * 16)); NN_TRY(A(&nn->y, n[0]));
  NN_TRY(A(&nn->dy, n[0])); NN_TRY(A(&nn->g0b, n[0] * 16));
  NN_TRY(A(&nn->gu0, n[0] * 32)); NN_TRY(A(&nn->g1, n[1] * 32)); NN_TRY(A(&nn->g1b, n[1] * 32));
  NN_TRY(A(&nn->gu1, n[1] * 64)); NN_TRY(A(&nn->g2, n[2] * 64)); NN_TRY(A(&nn->g2b, n[2] * 64));
  NN_TRY(A(&nn->gu2, n[2] * 64)); NN_TRY(A(&nn->g3b, n[3] * 64));
  size_t pc = HEAD_BLOCKS * 17;   // partial sums of the head's, then of each convolution's gradient
  for (int k = 0; k < NCONV; ++k) {
    int l = (k <= 3) ? k : 6 - k;   // resolution level of conv k's output
    size_t c = (size_t)wgrad_wgs(nn->lv[l], CIN_PAD[k], COUT[k]) * (27 * CIN_PAD[k] * COUT[k] + COUT[k]);
    pc = std::max(pc, c);
  }
  nn->part_cap = pc;
  NN_TRY(A(&nn->part, (long)pc));
  NN_TRY(A(&nn->lpart, 3L * B * 64));
  NN_TRY(A(&nn->loss, 1));
  return CPR_OK;
}

static void nn_free(cpr_nn* nn) {
  float* fs[] = {nn->theta, nn->m, nn->vv, nn->grad, nn->x3, nn->e0, nn->p1, nn->e1, nn->p2, nn->e2, nn->p3,
                 nn->e3, nn->a4, nn->d2, nn->a5, nn->d1, nn->a6, nn->d0, nn->y, nn->dy, nn->g0b,
                 nn->gu0, nn->g1, nn->g1b, nn->gu1, nn->g2, nn->g2b, nn->gu2, nn->g3b,
                 nn->part, nn->lpart, nn->loss};
  for (float* p : fs) dev_free(nn->mem, p);
  for (int k = 0; k < NCONV; ++k) {
    dev_free(nn->mem, nn->wf[k]);
    dev_free(nn->mem, nn->wb[k]);
  }
}

// Internal use by the solver's learned stage: x3's third channel is
// multiplied by *xscale (device scalar) as the network loads it.
int nn_infer(cpr_nn* nn, const float* x3, float* y, const double* xscale);
float* nn_output(cpr_nn* nn) { return nn->y; }

int nn_infer(cpr_nn* nn, const float* x3, float* y, const double* xscale) {
  long n0 = nn->lv[0].V;
  int rc = nn_forward_impl(nn, x3, 1, false, xscale);
  if (rc) return rc;
  if (y && y != nn->y) NN_TRY(hipMemcpyAsync(y, nn->y, n0 * sizeof(float), hipMemcpyDeviceToDevice, nn->stream));
  return CPR_OK;
}

void nn_set_stream(cpr_nn* nn, hipStream_t s) { nn->stream = s; }

extern "C" {

long long cpr_nn_num_params(void) { return nn_param_count(); }

int cpr_nn_create(int nx, int ny, int nz, int max_batch, void* stream, cpr_nn_t** out) {
  if (!out) return CPR_EINVAL;
  *out = nullptr;
  cpr_nn* nn = nullptr;
  try {
    nn = new cpr_nn();
  } catch (...) {
    return CPR_ENOMEM;
  }
  nn->mem = current_allocator();
  *out = nn;
  if (nx < 8 || ny < 8 || nz < 8 || nx % 8 || ny % 8 || nz % 8 || max_batch < 1 || max_batch > 64)
    return nn_err(nn, CPR_EINVAL, "grid dimensions must be multiples of 8 (>= 8), batch 1..64");
  if ((long)nx * ny * nz * max_batch > (1L << 28)) return nn_err(nn, CPR_EINVAL, "network input too large");
  nn->stream = (hipStream_t)stream;
  nn->max_batch = max_batch;
  for (int l = 0; l < 4; ++l) {
    nn->lv[l].nx = nx >> l; nn->lv[l].ny = ny >> l; nn->lv[l].nz = nz >> l;
    nn->lv[l].V = nn->lv[l].nx * nn->lv[l].ny * nn->lv[l].nz;
    nn->lv[l].batch = max_batch;
  }
  nn->P = nn_param_count();
  long o = 0;
  for (int k = 0; k < NCONV; ++k) {
    nn->off[k] = o;
    o += 27L * CIN[k] * COUT[k] + COUT[k];
  }
  nn->off[NCONV] = o;
  int rc = nn_alloc(nn);
  if (rc) return rc;
  NN_TRY(hipMemsetAsync(nn->theta, 0, nn->P * sizeof(float), nn->stream));
  NN_TRY(hipMemsetAsync(nn->m, 0, nn->P * sizeof(float), nn->stream));
  NN_TRY(hipMemsetAsync(nn->vv, 0, nn->P * sizeof(float), nn->stream));
  NN_TRY(hipStreamSynchronize(nn->stream));
  return CPR_OK;
}

void cpr_nn_destroy(cpr_nn_t* nn) {
  if (!nn) return;
  hipStreamSynchronize(nn->stream);
  nn_free(nn);
  delete nn;
}

const char* cpr_nn_last_error(const cpr_nn_t* nn) { return nn ? nn->err.c_str() : "null network"; }

int cpr_nn_set_params(cpr_nn_t* nn, const float* theta) {
  if (!nn || !theta) return CPR_EINVAL;
  NN_TRY(hipMemcpyAsync(nn->theta, theta, nn->P * sizeof(float), hipMemcpyHostToDevice, nn->stream));
  NN_TRY(hipMemsetAsync(nn->m, 0, nn->P * sizeof(float), nn->stream));
  NN_TRY(hipMemsetAsync(nn->vv, 0, nn->P * sizeof(float), nn->stream));
  nn->adam_step = 0;
  int rc = nn_refresh_frags(nn);
  if (rc) return rc;
  NN_TRY(hipStreamSynchronize(nn->stream));
  return CPR_OK;
}

int cpr_nn_get_adam(cpr_nn_t* nn, float* m, float* v, long long* step) {
  if (!nn || !m || !v || !step) return CPR_EINVAL;
  NN_TRY(hipMemcpyAsync(m, nn->m, nn->P * sizeof(float), hipMemcpyDeviceToHost, nn->stream));
  NN_TRY(hipMemcpyAsync(v, nn->vv, nn->P * sizeof(float), hipMemcpyDeviceToHost, nn->stream));
  NN_TRY(hipStreamSynchronize(nn->stream));
  *step = nn->adam_step;
  return CPR_OK;
}

int cpr_nn_set_adam(cpr_nn_t* nn, const float* m, const float* v, long long step) {
  if (!nn || !m || !v) return CPR_EINVAL;
  if (step < 0) return nn_err(nn, CPR_EINVAL, "negative Adam step count");
  NN_TRY(hipMemcpyAsync(nn->m, m, nn->P * sizeof(float), hipMemcpyHostToDevice, nn->stream));
  NN_TRY(hipMemcpyAsync(nn->vv, v, nn->P * sizeof(float), hipMemcpyHostToDevice, nn->stream));
  NN_TRY(hipStreamSynchronize(nn->stream));
  nn->adam_step = (long)step;
  return CPR_OK;
}

int cpr_nn_get_params(cpr_nn_t* nn, float* theta) {
  if (!nn || !theta) return CPR_EINVAL;
  NN_TRY(hipMemcpyAsync(theta, nn->theta, nn->P * sizeof(float), hipMemcpyDeviceToHost, nn->stream));
  NN_TRY(hipStreamSynchronize(nn->stream));
  return CPR_OK;
}

int cpr_nn_forward(cpr_nn_t* nn, const float* x, int batch, float* y) {
  if (!nn || !x || !y) return CPR_EINVAL;
  if (batch < 1 || batch > nn->max_batch) return nn_err(nn, CPR_EINVAL, "batch out of range");
  if (!nn->frags_valid) return nn_err(nn, CPR_EINVAL, "parameters not set");
  long n0 = (long)batch * nn->lv[0].V;
  // for the weight gradient, which may run after the caller has changed x
  NN_TRY(hipMemcpyAsync(nn->x3, x, n0 * 3 * sizeof(float), hipMemcpyDeviceToDevice, nn->stream));
  int rc = nn_forward_impl(nn, x, batch, true);
  if (rc) return rc;
  NN_TRY(hipMemcpyAsync(y, nn->y, n0 * sizeof(float), hipMemcpyDeviceToDevice, nn->stream));
  return CPR_OK;
}

int cpr_nn_infer(cpr_nn_t* nn, const float* x, float* y) {
  if (!nn || !x || !y) return CPR_EINVAL;
  if (!nn->frags_valid) return nn_err(nn, CPR_EINVAL, "parameters not set");
  return nn_infer(nn, x, y, nullptr);
}

int cpr_nn_backward(cpr_nn_t* nn, const float* dy, float* grad) {
  if (!nn || !dy || !grad) return CPR_EINVAL;
  if (nn->cur_batch < 1) return nn_err(nn, CPR_EINVAL, "no forward pass to differentiate");
  long n0 = (long)nn->cur_batch * nn->lv[0].V;
  NN_TRY(hipMemcpyAsync(nn->dy, dy, n0 * sizeof(float), hipMemcpyDeviceToDevice, nn->stream));
  int rc = nn_backward_impl(nn);
  if (rc) return rc;
  NN_TRY(hipMemcpyAsync(grad, nn->grad, nn->P * sizeof(float), hipMemcpyDeviceToDevice, nn->stream));
  return CPR_OK;
}

int cpr_nn_eval_loss(cpr_nn_t* nn, const float* x, const float* t, int batch, float* loss_out) {
  if (!nn || !x || !t || !loss_out) return CPR_EINVAL;
  if (batch < 1 || batch > nn->max_batch) return nn_err(nn, CPR_EINVAL, "batch out of range");
  if (!nn->frags_valid) return nn_err(nn, CPR_EINVAL, "parameters not set");
  hipStream_t s = nn->stream;
  const int V = nn->lv[0].V;
  long n0 = (long)batch * V;
  int rc = nn_forward_impl(nn, x, batch, false);
  if (rc) return rc;
  const int per = 64;
  loss_partial_kernel<<<batch * per, 256, 0, s>>>(V, per, nn->y, t, nn->lpart);
  loss_grad_kernel<<<div_up(n0, 256) < 1024 ? div_up(n0, 256) : 1024, 256, 0, s>>>(batch, V, per, nn->lpart, nn->y,
                                                                                  t, nn->dy, nn->loss);
  NN_TRY(hipMemcpyAsync(loss_out, nn->loss, sizeof(float), hipMemcpyDeviceToHost, s));
  NN_TRY(hipStreamSynchronize(s));
  return CPR_OK;
}

int cpr_nn_make_target(const double* e, long long n, double scale, float* t, void* stream) {
  if (!e || !t || n < 0 || !(scale > 0)) return CPR_EINVAL;
  if (n == 0) return CPR_OK;
  target_kernel<<<div_up(n, 256), 256, 0, (hipStream_t)stream>>>(n, e, 1.0 / scale, t);
  return hipGetLastError() == hipSuccess ? CPR_OK : CPR_EHIP;
}

int cpr_nn_train_step(cpr_nn_t* nn, const float* x, const float* t, int batch, float lr, float* loss_out) {
  if (!nn || !x || !t) return CPR_EINVAL;
  if (batch < 1 || batch > nn->max_batch || batch > 64) return nn_err(nn, CPR_EINVAL, "batch out of range");
  if (!nn->frags_valid) return nn_err(nn, CPR_EINVAL, "parameters not set");
  hipStream_t s = nn->stream;
  const int V = nn->lv[0].V;
  long n0 = (long)batch * V;
  NN_TRY(hipMemcpyAsync(nn->x3, x, n0 * 3 * sizeof(float), hipMemcpyDeviceToDevice, s));   // for the weight gradient
  int rc = nn_forward_impl(nn, x, batch, true);
  if (rc) return rc;
  const int per = 64;
  loss_partial_kernel<<<batch * per, 256, 0, s>>>(V, per, nn->y, t, nn->lpart);
  loss_grad_kernel<<<div_up(n0, 256) < 1024 ? div_up(n0, 256) : 1024, 256, 0, s>>>(batch, V, per, nn->lpart, nn->y,
                                                                                  t, nn->dy, nn->loss);
  rc = nn_backward_impl(nn);
  if (rc) return rc;
  nn->adam_step += 1;
  const float b1 = 0.9f, b2 = 0.999f;
  float c1 = 1.f / (1.f - powf(b1, (float)nn->adam_step));
  float c2 = 1.f / (1.f - powf(b2, (float)nn->adam_step));
  adam_kernel<<<div_up(nn->P, 256), 256, 0, s>>>(nn->P, lr, b1, b2, 1e-8f, c1, c2, nn->grad, nn->m, nn->vv,
                                                 nn->theta);
  rc = nn_refresh_frags(nn);
  if (rc) return rc;
  if (loss_out) {
    NN_TRY(hipMemcpyAsync(loss_out, nn->loss, sizeof(float), hipMemcpyDeviceToHost, s));
    NN_TRY(hipStreamSynchronize(s));
  }
  NN_TRY(hipGetLastError());
  return CPR_OK;
}

}  // extern "C"
