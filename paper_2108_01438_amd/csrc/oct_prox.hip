// Proximal operators of Sec. 2.2-2.3 (eq. (12)-(14), (16)), FP64 reductions
// and small elementwise helpers.
//
// * l1 (Psi = I): complex soft threshold z = v max(0, 1 - tau/|v|).
// * Haar: a multi-level orthonormal Haar pyramid over the depth and lateral
//   axes is local to blocks of 2^levels samples per axis.  Each thread takes a
//   2x2(x2) group, keeps its soft-thresholded detail coefficients in registers
//   and hands the low band one level up through LDS; the coarsest low band is
//   left untouched and the synthesis walks back down.
// * TV: isotropic complex TV (forward differences, zero at the last index)
//   by the fast gradient projection (FGP) of Beck and Teboulle on the dual,
//   x = v + tau div p.  The 2-D path runs all inner steps of a tile in LDS
//   (temporal blocking with a halo as wide as the dependence cone); the
//   3-D path runs a few inner steps per pass over memory, walking along y.
// All partial sums are per block in FP64 and summed in a fixed order.
#include "oct_fft.h"

#include <algorithm>

namespace {

__device__ double block_sum(double v, double* sh) {
#pragma unroll
  for (int o = 32; o > 0; o >>= 1) v += __shfl_xor(v, o);
  const int lane = threadIdx.x & 63, w = threadIdx.x >> 6;
  if (lane == 0) sh[w] = v;
  __syncthreads();
  double s = 0.0;
  if (threadIdx.x == 0) {
    const int nw = (blockDim.x + 63) >> 6;
    for (int i = 0; i < nw; ++i) s += sh[i];
  }
  return s;
}

__global__ void reduce_kernel(const double* __restrict__ p, int n, double* out, double scale, int accumulate) {
  __shared__ double sh[16];
  double acc = 0.0;
  for (int i = threadIdx.x; i < n; i += blockDim.x) acc += p[i];
  const double s = block_sum(acc, sh);
  if (threadIdx.x == 0) out[0] = accumulate ? out[0] + scale * s : scale * s;
}

__global__ void objective_kernel(const double* __restrict__ rp, int nr, const double* __restrict__ pp, int np,
                                 double lambda, double* out) {
  __shared__ double sh[16];
  double a = 0.0, b = 0.0;
  for (int i = threadIdx.x; i < nr; i += blockDim.x) a += rp[i];
  const double sa = block_sum(a, sh);
  __syncthreads();
  for (int i = threadIdx.x; i < np; i += blockDim.x) b += pp[i];
  const double sb = block_sum(b, sh);
  if (threadIdx.x == 0) out[0] = 0.5 * sa + lambda * sb;
}

__global__ void norm2_kernel(const float2* __restrict__ x, int64_t n, double* partial) {
  __shared__ double sh[16];
  double acc = 0.0;
  for (int64_t i = blockIdx.x * (int64_t)blockDim.x + threadIdx.x; i < n; i += (int64_t)gridDim.x * blockDim.x) {
    const float2 v = x[i];
    acc += (double)v.x * v.x + (double)v.y * v.y;
  }
  const double s = block_sum(acc, sh);
  if (threadIdx.x == 0) partial[blockIdx.x] = s;
}

__global__ void scale_inv_sqrt_kernel(const float2* __restrict__ x, float2* y, int64_t n, const double* sumsq) {
  // a zero vector stays zero (the power iteration on Phi = 0 gives L = 0)
  const double ss = sumsq[0];
  const float sc = ss > 0.0 ? (float)(1.0 / sqrt(ss)) : 0.f;
  for (int64_t i = blockIdx.x * (int64_t)blockDim.x + threadIdx.x; i < n; i += (int64_t)gridDim.x * blockDim.x)
    y[i] = cscale(x[i], sc);
}

// SplitMix64 (Steele, Lea and Flood 2014) as a counter generator.
__device__ __forceinline__ uint64_t splitmix64(uint64_t counter, uint64_t seed) {
  uint64_t z = seed + (counter + 1ull) * 0x9E3779B97F4A7C15ull;
  z = (z ^ (z >> 30)) * 0xBF58476D1CE4E5B9ull;
  z = (z ^ (z >> 27)) * 0x94D049BB133111EBull;
  return z ^ (z >> 31);
}
__device__ __forceinline__ double counter_uniform(uint64_t c, uint64_t seed) {
  return (double)(splitmix64(c, seed) >> 11) * 0x1.0p-52 - 1.0;
}

__global__ void uniform_kernel(float2* x, int64_t n, uint64_t seed) {
  for (int64_t i = blockIdx.x * (int64_t)blockDim.x + threadIdx.x; i < n; i += (int64_t)gridDim.x * blockDim.x)
    x[i] = make_float2((float)counter_uniform(2ull * i, seed), (float)counter_uniform(2ull * i + 1ull, seed));
}

__global__ void copy_kernel(const float2* __restrict__ x, float2* y, int64_t n) {
  for (int64_t i = blockIdx.x * (int64_t)blockDim.x + threadIdx.x; i < n; i += (int64_t)gridDim.x * blockDim.x)
    y[i] = x[i];
}

// y[b][i] = s_b x[b][i] for items of per_item elements (T = float or float2)
template <typename T>
__global__ void scale_items_kernel(const T* __restrict__ x, T* y, int64_t per_item, int64_t n, ItemScales sc) {
  for (int64_t i = blockIdx.x * (int64_t)blockDim.x + threadIdx.x; i < n; i += (int64_t)gridDim.x * blockDim.x) {
    const float f = sc.s[i / per_item];
    if constexpr (sizeof(T) == sizeof(float)) y[i] = x[i] * f;
    else y[i] = cscale(x[i], f);
  }
}

__global__ void zero_kernel(float2* y, int64_t n) {
  for (int64_t i = blockIdx.x * (int64_t)blockDim.x + threadIdx.x; i < n; i += (int64_t)gridDim.x * blockDim.x)
    y[i] = make_float2(0.f, 0.f);
}

// soft threshold by tau, then the modulus clipped to bound (the projection onto
// C; exact for l1 because the constrained problem stays radial per pixel)
__global__ void prox_l1_kernel(const float2* __restrict__ v, float2* z, int64_t n, float tau, float bound,
                               double* partial) {
  __shared__ double sh[16];
  double acc = 0.0;
  for (int64_t i = blockIdx.x * (int64_t)blockDim.x + threadIdx.x; i < n; i += (int64_t)gridDim.x * blockDim.x) {
    const float2 a = v[i];
    const float mag = sqrtf(a.x * a.x + a.y * a.y);
    const float sc = mag > tau ? fminf(1.f - tau / mag, bound / mag) : 0.f;
    const float2 r = make_float2(a.x * sc, a.y * sc);
    acc += (double)sqrtf(r.x * r.x + r.y * r.y);
    z[i] = r;
  }
  const double s = block_sum(acc, sh);
  if (threadIdx.x == 0 && partial) partial[blockIdx.x] = s;
}

// ---------------------------------------------------------------------------
// Haar pyramid on blocks of 2^LV per axis.  D = 2 (depth, x) or 3 (depth, x, y).
// A workgroup covers NBN blocks along depth; level-l groups are indexed
// (a, b, c) with a along depth fastest.
// ---------------------------------------------------------------------------
constexpr float RS2 = 0.70710678118654752440f;

// analysis of one group in place: index bits (depth, x, y), 0 = low
template <int D>
__device__ __forceinline__ void haar_fwd_group(float2* v) {
#pragma unroll
  for (int ax = 0; ax < D; ++ax) {
    const int bit = 1 << ax;
#pragma unroll
    for (int i = 0; i < (1 << D); ++i) {
      if (i & bit) continue;
      const float2 e = v[i], o = v[i | bit];
      v[i] = make_float2((e.x + o.x) * RS2, (e.y + o.y) * RS2);
      v[i | bit] = make_float2((e.x - o.x) * RS2, (e.y - o.y) * RS2);
    }
  }
}
template <int D>
__device__ __forceinline__ void haar_inv_group(float2* v) {
#pragma unroll
  for (int ax = D - 1; ax >= 0; --ax) {
    const int bit = 1 << ax;
#pragma unroll
    for (int i = 0; i < (1 << D); ++i) {
      if (i & bit) continue;
      const float2 lo = v[i], hi = v[i | bit];
      v[i] = make_float2((lo.x + hi.x) * RS2, (lo.y + hi.y) * RS2);
      v[i | bit] = make_float2((lo.x - hi.x) * RS2, (lo.y - hi.y) * RS2);
    }
  }
}

// soft threshold; with PART the modulus of the result joins the l1 partial sum
template <bool PART>
__device__ __forceinline__ float2 soft(float2 a, float tau, double& acc) {
  const float mag = sqrtf(a.x * a.x + a.y * a.y);
  const float sc = mag > tau ? 1.f - tau / mag : 0.f;
  const float2 r = make_float2(a.x * sc, a.y * sc);
  if (PART) acc += (double)sqrtf(r.x * r.x + r.y * r.y);
  return r;
}

// PART: also the per-block FP64 sums of |detail coefficients| (the penalty
// value), only when the caller asks for them
template <int D, int LV, int NBN, bool PART>
__global__ void __launch_bounds__(1024) haar_kernel(ProxGeom g, const float2* __restrict__ vin, float2* zout,
                                                    float tau, double* partial) {
  constexpr int NV = 1 << D;
  constexpr int BS = 1 << LV;                     // block side
  constexpr int GA0 = NBN * BS / 2;               // level-0 groups along depth
  constexpr int GB0 = BS / 2;                     // along x (and y)
  constexpr int GC0 = (D == 3) ? BS / 2 : 1;
  constexpr int NG0 = GA0 * GB0 * GC0;
  __shared__ float2 ll[2][NG0];
  __shared__ double sh[16];
  const int tid = threadIdx.x;
  const int Nz = g.Nz, Nx = g.Nx, Ny = g.Ny;
  // tile origin
  const int tz = Nz / (NBN * BS) + ((Nz % (NBN * BS)) ? 1 : 0);
  const int tx = Nx / BS;
  const int ty = (D == 3) ? Ny / BS : 1;
  int t = blockIdx.x;
  const int iz = t % tz; t /= tz;
  const int ix = t % tx; t /= tx;
  const int iy = t % ty; t /= ty;
  const int b = t;
  const int z0 = iz * NBN * BS, x0 = ix * BS, y0 = iy * BS;
  // a 2x2(x2) group at depth 2a, x 2bb, y 2c of the tile: its first element's
  // offset; the others lie 1 (depth), sx (x) and sy (y) further
  const int64_t sx = Nz, sy = (int64_t)Nx * Nz;
  auto group_off = [&](int a, int bb, int c) -> int64_t {
    return (((int64_t)b * Ny + y0 + 2 * c) * Nx + x0 + 2 * bb) * Nz + z0 + 2 * a;
  };
  auto elem_off = [&](int i) -> int64_t { return (i & 1) + ((i >> 1) & 1) * sx + ((i >> 2) & 1) * sy; };

  float2 det[LV][NV];
  double acc = 0.0;
  // level 0: load a 2x2(x2) group
  {
    if (tid < NG0) {
      const int a = tid % GA0, bb = (tid / GA0) % GB0, c = tid / (GA0 * GB0);
      float2 v[NV];
      const bool ok = z0 + 2 * a < Nz;
      const float2* __restrict__ src = vin + group_off(a, bb, c);
#pragma unroll
      for (int i = 0; i < NV; ++i) v[i] = ok ? src[elem_off(i)] : make_float2(0.f, 0.f);
      haar_fwd_group<D>(v);
#pragma unroll
      for (int i = 1; i < NV; ++i) det[0][i] = soft<PART>(v[i], tau, acc);
      ll[0][tid] = v[0];
    }
  }
  __syncthreads();
  // analysis up the pyramid
  int GA = GA0, GB = GB0, GC = GC0;
#pragma unroll
  for (int l = 1; l < LV; ++l) {
    const int nA = GA / 2, nB = GB / 2, nC = (D == 3) ? GC / 2 : 1;
    const int src = (l - 1) & 1, dstb = l & 1;
    if (tid < nA * nB * nC) {
      const int a = tid % nA, bb = (tid / nA) % nB, c = tid / (nA * nB);
      float2 v[NV];
#pragma unroll
      for (int i = 0; i < NV; ++i) {
        const int aa = 2 * a + (i & 1), b2 = 2 * bb + ((i >> 1) & 1), c2 = (D == 3) ? 2 * c + ((i >> 2) & 1) : 0;
        v[i] = ll[src][(c2 * GB + b2) * GA + aa];
      }
      haar_fwd_group<D>(v);
#pragma unroll
      for (int i = 1; i < NV; ++i) det[l][i] = soft<PART>(v[i], tau, acc);
      det[l][0] = v[0];   // coarsest low band kept (only used at l = LV-1)
      ll[dstb][tid] = v[0];
    }
    GA = nA; GB = nB; GC = nC;
    __syncthreads();
  }
  // synthesis down the pyramid (the top level keeps its low band)
#pragma unroll
  for (int l = LV - 1; l >= 1; --l) {
    // groups at level l: count GA*GB*GC (current sizes); parents write into ll[(l-1)&1]
    const int dstb = (l - 1) & 1;
    const int srcb = l & 1;
    if (tid < GA * GB * GC) {
      const int a = tid % GA, bb = (tid / GA) % GB, c = tid / (GA * GB);
      float2 v[NV];
      v[0] = (l == LV - 1) ? det[l][0] : ll[srcb][tid];
#pragma unroll
      for (int i = 1; i < NV; ++i) v[i] = det[l][i];
      haar_inv_group<D>(v);
      const int pA = GA * 2, pB = GB * 2;
#pragma unroll
      for (int i = 0; i < NV; ++i) {
        const int aa = 2 * a + (i & 1), b2 = 2 * bb + ((i >> 1) & 1), c2 = (D == 3) ? 2 * c + ((i >> 2) & 1) : 0;
        ll[dstb][(c2 * pB + b2) * pA + aa] = v[i];
      }
    }
    GA *= 2; GB *= 2; if (D == 3) GC *= 2;
    __syncthreads();
  }
  if (tid < NG0) {
    const int a = tid % GA0, bb = (tid / GA0) % GB0, c = tid / (GA0 * GB0);
    float2 v[NV];
    v[0] = ll[0][tid];
#pragma unroll
    for (int i = 1; i < NV; ++i) v[i] = det[0][i];
    haar_inv_group<D>(v);
    if (z0 + 2 * a < Nz) {
      float2* __restrict__ dst = zout + group_off(a, bb, c);
#pragma unroll
      for (int i = 0; i < NV; ++i) dst[elem_off(i)] = v[i];
    }
  }
  if (PART) {
    const double s = block_sum(acc, sh);
    if (tid == 0) partial[blockIdx.x] = s;
  }
}

template <int D, int LV> struct HaarCfg;
template <int LV> struct HaarCfg<2, LV> { static constexpr int NBN = (LV <= 3) ? (256 >> (2 * LV - 2)) / 1 * 1 : 1; };
template <int LV> struct HaarCfg<3, LV> { static constexpr int NBN = (LV <= 2) ? 8 : (LV == 3 ? 4 : 1); };

template <int D, int LV>
int haar_threads() {
  constexpr int BS = 1 << LV;
  constexpr int NBN = HaarCfg<D, LV>::NBN;
  return NBN * (BS / 2) * (BS / 2) * (D == 3 ? BS / 2 : 1);
}

template <int D, int LV>
int haar_blocks(const ProxGeom& g) {
  constexpr int BS = 1 << LV;
  constexpr int NBN = HaarCfg<D, LV>::NBN;
  const int tz = (g.Nz + NBN * BS - 1) / (NBN * BS);
  return tz * (g.Nx / BS) * ((D == 3) ? g.Ny / BS : 1) * g.B;
}

template <int D, int LV>
hipError_t haar_launch(const ProxGeom& g, const float2* v, float2* z, float tau, double* partial, hipStream_t s) {
  constexpr int NBN = HaarCfg<D, LV>::NBN;
  const int nt = haar_threads<D, LV>();
  const int nb = haar_blocks<D, LV>(g);
  if (partial)
    hipLaunchKernelGGL((haar_kernel<D, LV, NBN, true>), dim3(nb), dim3(nt < 64 ? 64 : nt), 0, s, g, v, z, tau, partial);
  else
    hipLaunchKernelGGL((haar_kernel<D, LV, NBN, false>), dim3(nb), dim3(nt < 64 ? 64 : nt), 0, s, g, v, z, tau,
                       partial);
  return hipGetLastError();
}

// ---------------------------------------------------------------------------
// TV by FGP, two passes per inner step (B-scans past the tile kernel's inner
// steps); the divergence and value kernels also serve volumes.
// strides: depth 1, x Nz, y Nx*Nz.  p, r: [nd][n] complex.
// ---------------------------------------------------------------------------
struct TvIdx {
  int Nz, Nx, Ny, nd;
  int64_t n;
  bool fast;              // n < 2^32: coordinates by 32-bit magic divisions
  FastDiv fz, fx, fy;
};

__device__ __forceinline__ void tv_coords(const TvIdx& d, int64_t i, int& iz, int& ix, int& iy) {
  if (d.fast) {
    const uint32_t u = (uint32_t)i, q1 = fdiv(u, d.fz), q2 = fdiv(q1, d.fx);
    iz = (int)(u - q1 * (uint32_t)d.Nz);
    ix = (int)(q1 - q2 * (uint32_t)d.Nx);
    iy = (int)(q2 - fdiv(q2, d.fy) * (uint32_t)d.Ny);
    return;
  }
  iz = (int)(i % d.Nz);
  const int64_t r = i / d.Nz;
  ix = (int)(r % d.Nx);
  iy = (int)((r / d.Nx) % d.Ny);
}

__device__ __forceinline__ float2 tv_div_at(const TvIdx& d, const float2* __restrict__ p, int64_t i, int iz,
                                            int ix, int iy) {
  float2 acc = make_float2(0.f, 0.f);
  const int64_t sx = d.Nz, sy = (int64_t)d.Nx * d.Nz;
  // depth
  if (iz < d.Nz - 1) acc = cadd(acc, p[i]);
  if (iz > 0) acc = csub(acc, p[i - 1]);
  // x
  if (ix < d.Nx - 1) acc = cadd(acc, p[d.n + i]);
  if (ix > 0) acc = csub(acc, p[d.n + i - sx]);
  if (d.nd == 3) {
    if (iy < d.Ny - 1) acc = cadd(acc, p[2 * d.n + i]);
    if (iy > 0) acc = csub(acc, p[2 * d.n + i - sy]);
  }
  return acc;
}

// out = P_C(v + tau div r), P_C the modulus clip to bound (+inf: none)
__global__ void tv_div_kernel(TvIdx d, const float2* __restrict__ v, const float2* __restrict__ r, float tau,
                              float bound, float2* out) {
  for (int64_t i = blockIdx.x * (int64_t)blockDim.x + threadIdx.x; i < d.n; i += (int64_t)gridDim.x * blockDim.x) {
    int iz, ix, iy;
    tv_coords(d, i, iz, ix, iy);
    const float2 dv = tv_div_at(d, r, i, iz, ix, iy);
    const float2 a = v[i];
    float2 x = make_float2(a.x + tau * dv.x, a.y + tau * dv.y);
    const float m2 = x.x * x.x + x.y * x.y;
    if (m2 > bound * bound) x = cscale(x, bound * rsqrtf(m2));
    out[i] = x;
  }
}

__global__ void tv_step_kernel(TvIdx d, const float2* __restrict__ dd, float2* r, float2* p, float step, float mom) {
  const int64_t sx = d.Nz, sy = (int64_t)d.Nx * d.Nz;
  for (int64_t i = blockIdx.x * (int64_t)blockDim.x + threadIdx.x; i < d.n; i += (int64_t)gridDim.x * blockDim.x) {
    int iz, ix, iy;
    tv_coords(d, i, iz, ix, iy);
    const float2 c = dd[i];
    float2 gz = (iz < d.Nz - 1) ? csub(dd[i + 1], c) : make_float2(0.f, 0.f);
    float2 gx = (ix < d.Nx - 1) ? csub(dd[i + sx], c) : make_float2(0.f, 0.f);
    float2 gy = make_float2(0.f, 0.f);
    if (d.nd == 3 && iy < d.Ny - 1) gy = csub(dd[i + sy], c);
    float2 pz = r[i], px = r[d.n + i], py = make_float2(0.f, 0.f);
    pz = make_float2(pz.x + step * gz.x, pz.y + step * gz.y);
    px = make_float2(px.x + step * gx.x, px.y + step * gx.y);
    float m2 = pz.x * pz.x + pz.y * pz.y + px.x * px.x + px.y * px.y;
    if (d.nd == 3) {
      py = r[2 * d.n + i];
      py = make_float2(py.x + step * gy.x, py.y + step * gy.y);
      m2 += py.x * py.x + py.y * py.y;
    }
    const float sc = m2 > 1.f ? 1.f / sqrtf(m2) : 1.f;
    pz = cscale(pz, sc);
    px = cscale(px, sc);
    py = cscale(py, sc);
    const float2 oz = p[i], ox = p[d.n + i];
    r[i] = make_float2(pz.x + mom * (pz.x - oz.x), pz.y + mom * (pz.y - oz.y));
    r[d.n + i] = make_float2(px.x + mom * (px.x - ox.x), px.y + mom * (px.y - ox.y));
    p[i] = pz;
    p[d.n + i] = px;
    if (d.nd == 3) {
      const float2 oy = p[2 * d.n + i];
      r[2 * d.n + i] = make_float2(py.x + mom * (py.x - oy.x), py.y + mom * (py.y - oy.y));
      p[2 * d.n + i] = py;
    }
  }
}

// Whole-wave lane shifts (DPP wave_shr:1 / wave_shl:1, zero filled at the
// wave edge): lane i receives lane i-1 (shr) or lane i+1 (shl).
__device__ __forceinline__ float lane_prev(float v) {
  return __int_as_float(__builtin_amdgcn_mov_dpp(__float_as_int(v), 0x138, 0xf, 0xf, true));
}
__device__ __forceinline__ float lane_next(float v) {
  return __int_as_float(__builtin_amdgcn_mov_dpp(__float_as_int(v), 0x130, 0xf, 0xf, true));
}

// ---------------------------------------------------------------------------
// 3-D TV by FGP, T inner steps per pass over memory.  A workgroup owns a
// 64 x 24 (depth x lateral) column of planes and walks along y; lane = depth
// sample, each of the 8 waves a strip of TV3_S lateral rows.  Stage t of the
// walk applies inner step t to the plane t behind the one just loaded, so
// only the last plane of each stage (r, d, p, v) is held, in registers.
// Depth neighbours move by lane shifts, strip edges through LDS (one barrier
// per stage and plane: the primal point's edge is read a plane later).  A
// step reaches one sample further in every direction: with a halo of T on
// every side of the tile and of the run of planes, the core is exact.
//
// The state is the dual of the last two steps (r = p + mom (p - p_prev) is
// formed on load), read from one pair of buffers and written to another:
// the pass reads 7 images (v, p, p_prev) and writes 6, whatever T is, where a
// step in two kernels (d = v + tau div r stored, then r and p updated) moved
// 18.  Memory bound (1.0 GB a pass of three steps at 1024 x 96 x 96 in 0.29 ms,
// with the halos 4.8 TB/s).  A prox of 10 steps: 2998 -> 1296 us there, 45.3 ->
// 17.1 ms at 2048 x 256 x 256, 176 -> 155 us at 256 x 40 x 45; with runs of at
// most 2 steps 1446 us, 20.8 ms and 149 us, of one 1744 us, 29.3 ms and 161 us.
// Three steps of 3 rows per thread fill the registers (242) and, with `hold`,
// the LDS (150 KB) of a workgroup per CU.
// ---------------------------------------------------------------------------
constexpr int TV3_S = 3;
constexpr int TV3_WAVES = 8;
constexpr int TV3_ROWS = TV3_S * TV3_WAVES;

// v or zero, by value (a conditional on two array elements would select between their addresses)
__device__ __forceinline__ float2 keep_if(bool c, float2 v) { return make_float2(c ? v.x : 0.f, c ? v.y : 0.f); }

// FIRST: one dual on entry (r = p; p itself zero when a.cold)
template <int T, bool FIRST>
__global__ void __launch_bounds__(TV3_WAVES * 64) tv3d_march_kernel(Tv3dArgs a) {
  __shared__ float2 xr[T][2][TV3_WAVES + 1][64];   // last r_x row of wave w in [w + 1]; [0] stays zero
  __shared__ float2 xd[T][2][TV3_WAVES + 1][64];   // first d row of wave w in [w]; [TV3_WAVES] stays zero
  // p and v of the plane a stage holds, each slot its own thread's (no barrier): too many for registers
  constexpr int HS = T > 1 ? T - 1 : 1;
  __shared__ float2 hold[HS][4][T > 1 ? TV3_S : 1][TV3_WAVES * 64];
  const int lane = threadIdx.x & 63, w = __builtin_amdgcn_readfirstlane(threadIdx.x >> 6);
  // consecutive tiles (depth, then lateral neighbours) on one XCD: their halos meet in its L2
  const int per = gridDim.x >> 3;
  const int bid = (int)(blockIdx.x & 7) * per + (int)(blockIdx.x >> 3);
  if (bid >= a.ntiles) return;
  const int tz = bid % a.ntz;
  int q = bid / a.ntz;
  const int tl = q % a.ntl;
  q /= a.ntl;
  const int ty = q % a.nty;
  const int b = q / a.nty;
  const int Nz = a.Nz, Nx = a.Nx, Ny = a.Ny;
  const int CZ = 64 - 2 * T, CL = TV3_ROWS - 2 * T;
  const int n = tz * CZ - T + lane;
  const int l0 = tl * CL - T + w * TV3_S;
  const int y0 = ty * a.CY, y1 = min(y0 + a.CY, Ny);
  const bool nin = n >= 0 && n < Nz;
  const bool zedge = n >= 0 && n < Nz - 1;                    // has a forward depth neighbour
  const bool zcore = nin && lane >= T && lane < 64 - T;
  const float tau = a.tau, step = a.step, bound = a.bound;
  for (int i = threadIdx.x; i < T * 2 * 64; i += TV3_WAVES * 64) {
    xr[i >> 7][(i >> 6) & 1][0][i & 63] = make_float2(0.f, 0.f);
    xd[i >> 7][(i >> 6) & 1][TV3_WAVES][i & 63] = make_float2(0.f, 0.f);
  }
  // byte offsets of the thread's samples inside a plane (clamped: loads of samples outside are masked)
  uint32_t off[TV3_S];
#pragma unroll
  for (int s = 0; s < TV3_S; ++s)
    off[s] = ((uint32_t)min(max(l0 + s, 0), Nx - 1) * (uint32_t)Nz + (uint32_t)min(max(n, 0), Nz - 1)) * 8u;
  auto at = [](const float2* plane, uint32_t o) __attribute__((always_inline)) {
    return *reinterpret_cast<const float2*>(reinterpret_cast<const char*>(plane) + o);
  };
  const int64_t plane = (int64_t)Nx * Nz;
  auto plane_off = [&](int y) __attribute__((always_inline)) { return ((int64_t)b * Ny + y) * plane; };

  // plane being loaded: v, p and p_prev (samples outside the image: a clamped
  // one's values, replaced by zero on use)
  float2 lv[TV3_S], lp[3][TV3_S], lo[FIRST ? 1 : 3][TV3_S];
  auto load_plane = [&](int y) __attribute__((always_inline)) {
    const int64_t po = plane_off(min(max(y, 0), Ny - 1));
#pragma unroll
    for (int s = 0; s < TV3_S; ++s) {
      lv[s] = at(a.v + po, off[s]);
#pragma unroll
      for (int c = 0; c < 3; ++c) {
        lp[c][s] = at(a.p[c] + po, off[s]);
        if constexpr (!FIRST) lo[c][s] = at(a.po[c] + po, off[s]);
      }
    }
  };

  // per stage, the previous plane's r and d (and in `hold` its p and v)
  float2 cr[T][3][TV3_S], cd[T][TV3_S];
#pragma unroll
  for (int t = 0; t < T; ++t)
#pragma unroll
    for (int s = 0; s < TV3_S; ++s) {
      cd[t][s] = make_float2(0.f, 0.f);
#pragma unroll
      for (int c = 0; c < 3; ++c) cr[t][c][s] = make_float2(0.f, 0.f);
      if (t < T - 1)
#pragma unroll
        for (int c = 0; c < 4; ++c) hold[t][c][s][threadIdx.x] = make_float2(0.f, 0.f);
    }

  load_plane(y0 - T);
  int par = 0;
  for (int Y = y0 - T; Y < y1 + T; ++Y, par ^= 1) {
    float2 rn[3][TV3_S], pn[3][TV3_S], vn[TV3_S];
    const bool yin = Y >= 0 && Y < Ny;
#pragma unroll
    for (int s = 0; s < TV3_S; ++s) {
      const bool in = nin && yin && l0 + s >= 0 && l0 + s < Nx;
      vn[s] = keep_if(in, lv[s]);
#pragma unroll
      for (int c = 0; c < 3; ++c) {
        pn[c][s] = keep_if(FIRST ? in && !a.cold : in, lp[c][s]);
        rn[c][s] = pn[c][s];
        if constexpr (!FIRST) {
          const float2 o = keep_if(in, lo[c][s]);
          rn[c][s] = make_float2(pn[c][s].x + a.m0 * (pn[c][s].x - o.x), pn[c][s].y + a.m0 * (pn[c][s].y - o.y));
        }
      }
    }
    if (Y + 1 < y1 + T) load_plane(Y + 1);
#pragma unroll
    for (int t = 0; t < T; ++t) {
      // incoming: r_t, p_t, v of plane yt; held: r_t, d_t, p_t, v of plane yt - 1
      const int yt = Y - t;
      const bool ye = yt >= 0 && yt < Ny - 1, yem = yt - 1 >= 0 && yt - 1 < Ny - 1;   // forward y edges
      auto rx_in = [&](int s) __attribute__((always_inline)) {   // r_x where it has an edge
        const int l = l0 + s;
        return keep_if(l >= 0 && l < Nx - 1, rn[1][s]);
      };
      xr[t][par][w + 1][lane] = rx_in(TV3_S - 1);
      __syncthreads();
      float2 d[TV3_S];
#pragma unroll
      for (int s = 0; s < TV3_S; ++s) {
        const float2 rz = keep_if(zedge, rn[0][s]);
        const float2 rx = rx_in(s);
        float2 rxp;
        if (s > 0) rxp = rx_in(s - 1);
        else rxp = xr[t][par][w][lane];
        const float2 ry = keep_if(ye, rn[2][s]), ryp = keep_if(yem, cr[t][2][s]);
        const float dx = rz.x - lane_prev(rz.x) + rx.x - rxp.x + ry.x - ryp.x;
        const float dy = rz.y - lane_prev(rz.y) + rx.y - rxp.y + ry.y - ryp.y;
        float2 x = make_float2(fmaf(tau, dx, vn[s].x), fmaf(tau, dy, vn[s].y));
        const float m2 = x.x * x.x + x.y * x.y;
        if (m2 > bound * bound) x = cscale(x, bound * rsqrtf(m2));
        d[s] = x;
      }
      xd[t][par][w][lane] = d[0];   // read with the next plane
      // the held plane's step; the last two steps' duals leave for memory: plane
      // Y - T of the last, Y - T + 1 of the one before
      const int yo = yt - 1;
      float2* const* out = t == T - 1 ? a.out : a.out_prev;
      const bool store = t >= T - 2 && out[0] && yo >= y0 && yo < y1;
      const int64_t po = plane_off(yo);
#pragma unroll
      for (int s = 0; s < TV3_S; ++s) {
        const int l = l0 + s;
        const float2 c = cd[t][s];
        float2 dl;
        if (s < TV3_S - 1) dl = cd[t][s + 1];
        else dl = xd[t][par ^ 1][w + 1][lane];
        const float2 nz = make_float2(lane_next(c.x), lane_next(c.y));
        const float2 gz = keep_if(zedge, csub(nz, c)), gx = keep_if(l >= 0 && l < Nx - 1, csub(dl, c)),
                     gy = keep_if(yem, csub(d[s], c));
        float2 p1[3];
        p1[0] = make_float2(fmaf(step, gz.x, cr[t][0][s].x), fmaf(step, gz.y, cr[t][0][s].y));
        p1[1] = make_float2(fmaf(step, gx.x, cr[t][1][s].x), fmaf(step, gx.y, cr[t][1][s].y));
        p1[2] = make_float2(fmaf(step, gy.x, cr[t][2][s].x), fmaf(step, gy.y, cr[t][2][s].y));
        const float m2 = p1[0].x * p1[0].x + p1[0].y * p1[0].y + p1[1].x * p1[1].x + p1[1].y * p1[1].y +
                         (p1[2].x * p1[2].x + p1[2].y * p1[2].y);
        const float sc = m2 > 1.f ? __builtin_amdgcn_rsqf(m2) : 1.f;
        const int row = w * TV3_S + s;
        const bool st = store && zcore && row >= T && row < TV3_ROWS - T && l < Nx;
#pragma unroll
        for (int k = 0; k < 3; ++k) {
          p1[k] = cscale(p1[k], sc);
          if (t >= T - 2 && st)
            *reinterpret_cast<float2*>(reinterpret_cast<char*>(out[k] + po) + off[s]) = p1[k];
          // hold the incoming plane; the next stage takes the finished one
          cr[t][k][s] = rn[k][s];
          if (t < T - 1) {
            const float2 ph = hold[t][k][s][threadIdx.x];
            hold[t][k][s][threadIdx.x] = pn[k][s];
            rn[k][s] = make_float2(p1[k].x + a.mom[t] * (p1[k].x - ph.x), p1[k].y + a.mom[t] * (p1[k].y - ph.y));
            pn[k][s] = p1[k];
          }
        }
        if (t < T - 1) {
          const float2 vh = hold[t][3][s][threadIdx.x];
          hold[t][3][s][threadIdx.x] = vn[s];
          vn[s] = vh;
        }
        cd[t][s] = d[s];
        __builtin_amdgcn_sched_barrier(0);   // one row at a time: interleaved rows would not fit the registers
      }
    }
  }
}

__global__ void tv_value_kernel(TvIdx d, const float2* __restrict__ z, double* partial) {
  __shared__ double sh[16];
  const int64_t sx = d.Nz, sy = (int64_t)d.Nx * d.Nz;
  double acc = 0.0;
  for (int64_t i = blockIdx.x * (int64_t)blockDim.x + threadIdx.x; i < d.n; i += (int64_t)gridDim.x * blockDim.x) {
    int iz, ix, iy;
    tv_coords(d, i, iz, ix, iy);
    const float2 c = z[i];
    float m2 = 0.f;
    if (iz < d.Nz - 1) { const float2 g = csub(z[i + 1], c); m2 += g.x * g.x + g.y * g.y; }
    if (ix < d.Nx - 1) { const float2 g = csub(z[i + sx], c); m2 += g.x * g.x + g.y * g.y; }
    if (d.nd == 3 && iy < d.Ny - 1) { const float2 g = csub(z[i + sy], c); m2 += g.x * g.x + g.y * g.y; }
    acc += (double)sqrtf(m2);
  }
  const double s = block_sum(acc, sh);
  if (threadIdx.x == 0 && partial) partial[blockIdx.x] = s;
}

// ---------------------------------------------------------------------------
// 2-D TV by FGP with every inner step of a tile on chip.  Lane = depth sample
// (64 per wave, coalesced), each thread owns a strip of S lateral samples in
// registers, WAVES waves side by side laterally: a 64 x (WAVES S) loaded tile.
// Depth neighbours move by lane shuffles, lateral neighbours inside a strip are
// registers and across strips go through LDS.  One inner step reaches one
// sample further in every direction: with a halo of n_inner + 1 below (which z
// = v + tau div p reads) and n_inner above the dual is exact on the core; TV(z),
// where it is wanted, takes one more above.
// Bound: the vector units (1.7 us per step and 256 tiles of 64 x 128) and the
// loads and stores (about 15 us per 256 such tiles), in series when one
// workgroup fills a CU.  Two workgroups of eight waves per CU overlap them but
// spend more on halos (core 43 x 51 of 64 x 72 at ten steps, 43 x 107 of 64 x
// 128); strips of nine are the longest that gain (ten: 58.6 us, eight: 62.1).
// Two steps per turn of the loop spare the copies that swap the registers of r
// and P (53.0 us on 2048 x 1000), but spill 8 to 64 bytes per lane ahead of it:
// not used.  Ten steps on 2048 x 1000: 62.8 -> 54.9 us; on 8 x 1024 x 512: 131 ->
// 115 us.
// ---------------------------------------------------------------------------
constexpr int TV_S1 = 9, TV_W1 = 8;
constexpr int TV_S2 = 8, TV_W2 = 16;

// The dual is kept zero wherever its component has no forward edge (last
// index along that axis, and every sample outside the image).  The step of
// such a component is zero too, so it stays zero, and the divergence needs
// no boundary tests: (div p)_i = p_i - p_{i-1} along each axis.
// BOUND: the constrained FGP of Beck and Teboulle, the primal point projected
// onto C = {|x_i| <= bound} in every step and at the end.
template <int S, int WAVES, bool BOUND>
__global__ void __launch_bounds__(WAVES * 64, 4) tv2d_tile_kernel(Tv2dArgs a) {
  // strip-edge exchange rows: wave w publishes its last column in xr[w + 1]
  // and its first in xd[w]; xr[0] and xd[WAVES] stay zero, so every read
  // is unconditional
  __shared__ float2 xr[WAVES + 1][64];
  __shared__ float2 xd[WAVES + 1][64];
  __shared__ double sh[16];
  // the wave index is uniform: strip positions and lateral edge weights stay in
  // scalar registers
  const int lane = threadIdx.x & 63, w = __builtin_amdgcn_readfirstlane(threadIdx.x >> 6);
  // Consecutive blocks go to the eight XCDs in turn; tile numbers are dealt
  // so that each XCD runs a run of consecutive tiles (depth neighbours, whose
  // halos overlap, share its L2).  The grid is padded to a multiple of 8.
  const int per = gridDim.x >> 3;
  const int bid = (int)(blockIdx.x & 7) * per + (int)(blockIdx.x >> 3);
  if (bid >= a.ntiles) return;
  const int tz = bid % a.ntz;
  const int tl = (bid / a.ntz) % a.ntl;
  const int b = bid / (a.ntz * a.ntl);
  const int Nz = a.Nz, Nx = a.Nx, H = a.H;
  const int cz0 = tz * a.CZ, cl0 = tl * a.CL;
  const int n = cz0 - H + lane;
  const int l0 = cl0 - H + w * S;
  const bool nin = (n >= 0 && n < Nz);
  const bool zedge = (n >= 0 && n < Nz - 1);
  const int64_t ib = (int64_t)b * Nx * Nz;
  const int64_t N = a.n_total;
  const float tau = a.tau, step = a.step, bound = a.bound;
  const float sz = zedge ? step : 0.f;
  auto proj = [&](float2 x) __attribute__((always_inline)) {
    if (!BOUND) return x;
    const float sc = fminf(1.f, bound * __builtin_amdgcn_rsqf(x.x * x.x + x.y * x.y));
    return cscale(x, sc);
  };
  if (w == 0) xr[0][lane] = make_float2(0.f, 0.f);
  if (w == WAVES - 1) xd[WAVES][lane] = make_float2(0.f, 0.f);

  // FGP state per pixel: the extrapolated dual r and the previous dual P,
  // kept pre-multiplied by the momentum of the step that consumes it, so that
  // r = (1 + mom_k) p_k - mom_k p_{k-1} is one fused multiply-add per
  // component (mom after the last step is 1: P ends as the plain dual).  P is
  // updated in place: each pixel reads its old P before writing the new one.
  float2 v[S], Pz[S], Pl[S], rz[S], rl[S];
  uint32_t lfwd = 0;   // bit s: strip row s has a lateral forward edge
  const float mom0 = a.mom[0];
#pragma unroll
  for (int s = 0; s < S; ++s) {
    const int l = l0 + s;
    const bool in = nin && l >= 0 && l < Nx;
    const bool ledge = l >= 0 && l < Nx - 1;
    lfwd |= ledge ? 1u << s : 0u;
    const int64_t idx = ib + (int64_t)l * Nz + n;
    v[s] = in ? a.v[idx] : make_float2(0.f, 0.f);
    rz[s] = (in && zedge && a.pin) ? a.pin[idx] : make_float2(0.f, 0.f);
    rl[s] = (in && ledge && a.pin) ? a.pin[N + idx] : make_float2(0.f, 0.f);
    Pz[s] = cscale(rz[s], mom0);
    Pl[s] = cscale(rl[s], mom0);
  }
  for (int k = 0; k < a.n_inner; ++k) {
    asm volatile("" : "+s"(lfwd));   // weights chosen by the scalar unit in each step, not kept in S registers
    const float mom1 = 1.f + a.mom[k];
    const float mnext = a.mom[k + 1];
    xr[w + 1][lane] = rl[S - 1];
    __syncthreads();
    float2 d[S];
#pragma unroll
    for (int s = 0; s < S; ++s) {
      const float2 lp = (s > 0) ? rl[s - 1] : xr[w][lane];
      const float dx = (rz[s].x - lane_prev(rz[s].x)) + (rl[s].x - lp.x);
      const float dy = (rz[s].y - lane_prev(rz[s].y)) + (rl[s].y - lp.y);
      d[s] = proj(make_float2(fmaf(tau, dx, v[s].x), fmaf(tau, dy, v[s].y)));
    }
    xd[w][lane] = d[0];
    __syncthreads();
#pragma unroll
    for (int s = 0; s < S; ++s) {
      const float2 dl = (s < S - 1) ? d[s + 1] : xd[w + 1][lane];
      const float2 qz = make_float2(fmaf(sz, lane_next(d[s].x) - d[s].x, rz[s].x),
                                    fmaf(sz, lane_next(d[s].y) - d[s].y, rz[s].y));
      const float sl = (lfwd >> s) & 1u ? step : 0.f;
      const float2 ql = make_float2(fmaf(sl, dl.x - d[s].x, rl[s].x), fmaf(sl, dl.y - d[s].y, rl[s].y));
      const float m2 = qz.x * qz.x + qz.y * qz.y + ql.x * ql.x + ql.y * ql.y;
      // projection onto |p| <= 1: 1/sqrt(m2) when m2 > 1, else 1 (m2 = 0 included)
      const float sc = fminf(1.f, __builtin_amdgcn_rsqf(m2));
      const float ca = mom1 * sc, cb = mnext * sc;
      rz[s] = make_float2(fmaf(ca, qz.x, -Pz[s].x), fmaf(ca, qz.y, -Pz[s].y));
      rl[s] = make_float2(fmaf(ca, ql.x, -Pl[s].x), fmaf(ca, ql.y, -Pl[s].y));
      Pz[s] = cscale(qz, cb);
      Pl[s] = cscale(ql, cb);
    }
  }
  // z = v + tau div p  (P holds p after the last step)
  xr[w + 1][lane] = Pl[S - 1];
  __syncthreads();
  float2 z[S];
#pragma unroll
  for (int s = 0; s < S; ++s) {
    const float2 lp = (s > 0) ? Pl[s - 1] : xr[w][lane];
    const float dx = (Pz[s].x - lane_prev(Pz[s].x)) + (Pl[s].x - lp.x);
    const float dy = (Pz[s].y - lane_prev(Pz[s].y)) + (Pl[s].y - lp.y);
    z[s] = proj(make_float2(fmaf(tau, dx, v[s].x), fmaf(tau, dy, v[s].y)));
  }
  const bool zcore = nin && n >= cz0 && n < cz0 + a.CZ;
  if (a.partial) {   // TV(z) on the core as well, when the caller asks for it
    xd[w][lane] = z[0];
    __syncthreads();
    double acc = 0.0;
#pragma unroll
    for (int s = 0; s < S; ++s) {
      const int l = l0 + s;
      const float dnx = lane_next(z[s].x), dny = lane_next(z[s].y);
      const float2 zl = (s < S - 1) ? z[s + 1] : xd[w + 1][lane];
      if (zcore && l >= cl0 && l < cl0 + a.CL && l < Nx) {
        float m2 = 0.f;
        if (zedge) m2 += (dnx - z[s].x) * (dnx - z[s].x) + (dny - z[s].y) * (dny - z[s].y);
        if (l < Nx - 1) m2 += (zl.x - z[s].x) * (zl.x - z[s].x) + (zl.y - z[s].y) * (zl.y - z[s].y);
        acc += (double)sqrtf(m2);
      }
    }
    const double sum = block_sum(acc, sh);
    if (threadIdx.x == 0) a.partial[bid] = sum;
  }
#pragma unroll
  for (int s = 0; s < S; ++s) {
    const int l = l0 + s;
    if (zcore && l >= cl0 && l < cl0 + a.CL && l < Nx) {
      const int64_t idx = ib + (int64_t)l * Nz + n;
      a.z[idx] = z[s];
      a.pout[idx] = Pz[s];
      a.pout[N + idx] = Pl[s];
    }
  }
}

int grid_for(int64_t n, int nt) {
  int64_t b = (n + nt - 1) / nt;
  if (b > 2048) b = 2048;
  if (b < 1) b = 1;
  return (int)b;
}

}  // namespace

// ---------------------------------------------------------------------------
// launchers
// ---------------------------------------------------------------------------
hipError_t launch_reduce_sum(const double* partial, int n, double* out, double scale, int accumulate,
                             hipStream_t s) {
  hipLaunchKernelGGL(reduce_kernel, dim3(1), dim3(1024), 0, s, partial, n, out, scale, accumulate);
  return hipGetLastError();
}

hipError_t launch_objective(const double* rp, int nr, const double* pp, int np, double lambda, double* out,
                            hipStream_t s) {
  hipLaunchKernelGGL(objective_kernel, dim3(1), dim3(1024), 0, s, rp, nr, pp, np, lambda, out);
  return hipGetLastError();
}

hipError_t launch_norm2_partial(const float2* x, int64_t n, double* partial, int nblocks, hipStream_t s) {
  hipLaunchKernelGGL(norm2_kernel, dim3(nblocks), dim3(256), 0, s, x, n, partial);
  return hipGetLastError();
}

hipError_t launch_scale_by_inv_sqrt(const float2* x, float2* y, int64_t n, const double* sumsq, hipStream_t s) {
  hipLaunchKernelGGL(scale_inv_sqrt_kernel, dim3(grid_for(n, 256)), dim3(256), 0, s, x, y, n, sumsq);
  return hipGetLastError();
}

hipError_t launch_fill_counter_uniform(float2* x, int64_t n, uint64_t seed, hipStream_t s) {
  hipLaunchKernelGGL(uniform_kernel, dim3(grid_for(n, 256)), dim3(256), 0, s, x, n, seed);
  return hipGetLastError();
}

hipError_t launch_copy(const float2* x, float2* y, int64_t n, hipStream_t s) {
  hipLaunchKernelGGL(copy_kernel, dim3(grid_for(n, 256)), dim3(256), 0, s, x, y, n);
  return hipGetLastError();
}

hipError_t launch_scale_items(const float* x, float* y, int64_t per_item, int items, const ItemScales& sc,
                              hipStream_t s) {
  const int64_t n = per_item * items;
  hipLaunchKernelGGL(scale_items_kernel<float>, dim3(grid_for(n, 256)), dim3(256), 0, s, x, y, per_item, n, sc);
  return hipGetLastError();
}

hipError_t launch_scale_items(const float2* x, float2* y, int64_t per_item, int items, const ItemScales& sc,
                              hipStream_t s) {
  const int64_t n = per_item * items;
  hipLaunchKernelGGL(scale_items_kernel<float2>, dim3(grid_for(n, 256)), dim3(256), 0, s, x, y, per_item, n, sc);
  return hipGetLastError();
}

hipError_t launch_zero(float2* x, int64_t n, hipStream_t s) {
  hipLaunchKernelGGL(zero_kernel, dim3(grid_for(n, 256)), dim3(256), 0, s, x, n);
  return hipGetLastError();
}

hipError_t launch_prox_l1(const float2* v, float2* z, int64_t n, float tau, float bound, double* partial,
                          int nblocks, hipStream_t s) {
  hipLaunchKernelGGL(prox_l1_kernel, dim3(nblocks), dim3(256), 0, s, v, z, n, tau, bound, partial);
  return hipGetLastError();
}

int haar_partials(const ProxGeom& g, int levels) {
  if (g.lateral_dims == 1) {
    switch (levels) {
      case 1: return haar_blocks<2, 1>(g);
      case 2: return haar_blocks<2, 2>(g);
      case 3: return haar_blocks<2, 3>(g);
      case 4: return haar_blocks<2, 4>(g);
      case 5: return haar_blocks<2, 5>(g);
    }
  } else {
    switch (levels) {
      case 1: return haar_blocks<3, 1>(g);
      case 2: return haar_blocks<3, 2>(g);
      case 3: return haar_blocks<3, 3>(g);
      case 4: return haar_blocks<3, 4>(g);
    }
  }
  return -1;
}

hipError_t launch_prox_haar(const ProxGeom& g, int levels, const float2* v, float2* z, float tau, double* partial,
                            hipStream_t s) {
  if (g.lateral_dims == 1) {
    switch (levels) {
      case 1: return haar_launch<2, 1>(g, v, z, tau, partial, s);
      case 2: return haar_launch<2, 2>(g, v, z, tau, partial, s);
      case 3: return haar_launch<2, 3>(g, v, z, tau, partial, s);
      case 4: return haar_launch<2, 4>(g, v, z, tau, partial, s);
      case 5: return haar_launch<2, 5>(g, v, z, tau, partial, s);
    }
  } else {
    switch (levels) {
      case 1: return haar_launch<3, 1>(g, v, z, tau, partial, s);
      case 2: return haar_launch<3, 2>(g, v, z, tau, partial, s);
      case 3: return haar_launch<3, 3>(g, v, z, tau, partial, s);
      case 4: return haar_launch<3, 4>(g, v, z, tau, partial, s);
    }
  }
  return hipErrorInvalidValue;
}

size_t tv_work_elems(const ProxGeom& g) {
  const int nd = g.lateral_dims + 1;
  const int64_t n = (int64_t)g.B * g.Ny * g.Nx * g.Nz;
  return (size_t)n * (size_t)(1 + nd);     // d, r of the general path
}

static bool tv_tiled(const ProxGeom& g, int n_inner) {
  return g.lateral_dims == 1 && n_inner >= 1 && n_inner <= TV_MAX_TILED_INNER;
}

// Tiles of the 2-D step: core sizes and counts.  value: TV(z) is wanted too,
// which reads z one sample past the core.
struct Tv2dTiles {
  int waves, CZ, CL, ntz, ntl;
};

// Times (us) of tiles and n inner steps from a warm dual, by rounds of workgroups
// over the 256 CUs: two of the 64 x 72 tiles share a CU (one loads and stores
// while the other computes), one of the 64 x 128 fills it.  Past the first round
// the next workgroups overlap the last ones'.  Fitted to 11984 sizes and step
// counts; the choice costs 0.2 % on average against the better tile of each (a
// rule on the loaded samples, 3.4 %).  Measured, small against large (us): 2048 x
// 1000 with 10 steps 54.9 / 62.8, 16 steps 138 / 124, 20 steps 259 / 222; 8 x 1024
// x 512 with 10 steps 115 / 131; 512 x 64 with 10 steps 19.5 / 25.9; where the
// small tiles just miss a round (546 and 528 on 512 places) 1458 x 540 with 14
// steps 61 / 46, 600 x 1890 with 10 steps 40 / 29.
static double tv2d_us_small(int64_t tiles, int n) {
  const double one = 7.8 + 1.15 * n, two = 5.8 + 2.28 * n;   // a round of one and of two workgroups per CU
  if (tiles <= 256) return one;
  if (tiles <= 512) return two;
  return std::max(two + 0.62 * one, 0.8 * (double)tiles / 512.0 * two + 0.44 * one);
}

static double tv2d_us_large(int64_t tiles, int n) {
  const double one = 9.7 + 1.91 * n;
  return tiles <= 256 ? one : std::max(1.86 * one, 0.94 * (double)tiles / 256.0 * one + 0.2 * one);
}

static Tv2dTiles tv2d_tiles(const ProxGeom& g, int n_inner, bool value) {
  const int halo = 2 * n_inner + (value ? 2 : 1);
  auto make = [&](int strip, int waves) {
    Tv2dTiles t;
    t.waves = waves;
    t.CZ = 64 - halo;
    t.CL = strip * waves - halo;
    t.ntz = (g.Nz + t.CZ - 1) / t.CZ;
    t.ntl = (g.Nx + t.CL - 1) / t.CL;
    return t;
  };
  const Tv2dTiles t1 = make(TV_S1, TV_W1), t2 = make(TV_S2, TV_W2);
  const int64_t n1 = (int64_t)t1.ntz * t1.ntl * g.B, n2 = (int64_t)t2.ntz * t2.ntl * g.B;
  return 1.02 * tv2d_us_small(n1, n_inner) <= tv2d_us_large(n2, n_inner) ? t1 : t2;
}

template <int ST, int WAVES>
static void tv2d_launch(const Tv2dArgs& a, int nb, float bound, hipStream_t s) {
  if (bound < INFINITY) hipLaunchKernelGGL((tv2d_tile_kernel<ST, WAVES, true>), dim3(nb), dim3(WAVES * 64), 0, s, a);
  else hipLaunchKernelGGL((tv2d_tile_kernel<ST, WAVES, false>), dim3(nb), dim3(WAVES * 64), 0, s, a);
}

int tv_partials(const ProxGeom& g, int n_inner) {
  if (tv_tiled(g, n_inner)) {
    const Tv2dTiles t = tv2d_tiles(g, n_inner, true);
    return t.ntz * t.ntl * g.B;
  }
  const int64_t n = (int64_t)g.B * g.Ny * g.Nx * g.Nz;
  return grid_for(n, 256);
}

// Planes along y per workgroup (CY) and runs of planes (nty): the pass takes
// rounds of workgroups over the 256 CUs (one resident per CU), each CY planes
// and 2 T of halo long.
struct Tv3dSplit {
  int ntz, ntl, nty, CY;
  int64_t cols, rounds;
};

static Tv3dSplit tv3d_split(const ProxGeom& g, int T) {
  Tv3dSplit s{};
  const int CZ = 64 - 2 * T, CL = TV3_ROWS - 2 * T;
  s.ntz = (g.Nz + CZ - 1) / CZ;
  s.ntl = (g.Nx + CL - 1) / CL;
  s.cols = (int64_t)s.ntz * s.ntl * g.B;
  int64_t best = INT64_MAX;
  for (int n = 1; n <= g.Ny; ++n) {
    const int cy = (g.Ny + n - 1) / n, nty = (g.Ny + cy - 1) / cy;
    const int64_t rounds = (s.cols * nty + 255) / 256, cost = rounds * (cy + 2 * T + 2);
    if (cost < best) {
      best = cost;
      s.CY = cy;
      s.nty = nty;
      s.rounds = rounds;
    }
  }
  return s;
}

static int tv3d_passes(int n_inner) { return (n_inner + TV3_MAX_T - 1) / TV3_MAX_T; }
static int tv3d_pass_steps(int left, int passes_left) {   // as even as possible
  return (left + passes_left - 1) / passes_left;
}

// Whether a volume takes the walk along y (its passes by steps in split, zero on
// entry) or two kernels per step (d = v + tau div r stored, then r and p).  A
// pass of the walk is a chain of planes (2.0, 3.5 and 4.7 us each with 1, 2 and 3
// steps; 1.9, 2.7 and 3.8 in the first pass, which reads one dual), three and
// more of them halo, however small the volume.  The two kernels take about 6.5 us
// a step, as fast as the host launches them, until the memory traffic shows (23
// us per million samples), and copy the dual first.  So small volumes, and those
// a few rows wide (an empty tile costs as much), keep the two kernels for more
// than two steps.  Fitted to 1425 volumes with 2 to 20 steps; the choice costs
// 0.1 % on average against the better way of each and more than 4 % against the
// two kernels in 49 of 8550.  Measured, walk against two kernels, 10 steps (us):
// 128 x 16 x 16 103 / 88, 2048 x 8 x 8 125 / 87, 1024 x 4 x 100 208 / 148, 1024 x
// 1 x 256 359 / 120, 512 x 20 x 20 120 / 104; 256 x 40 x 45 137 / 149, 512 x 32 x
// 32 146 / 168, 512 x 64 x 64 274 / 556; three steps on 128 x 16 x 16 31 / 28 to
// 37.
static bool tv3d_walks(const ProxGeom& g, int n_inner, Tv3dSplit* split) {
  static const double first_us[TV3_MAX_T + 1] = {0, 1.9, 2.7, 3.8}, plane_us[TV3_MAX_T + 1] = {0, 2.0, 3.5, 4.7};
  const double mpx = 1e-6 * (double)g.B * g.Ny * g.Nx * g.Nz;
  const double two = std::max(4.7, 20.0 * mpx) + n_inner * std::max(6.5, 6.0 + 23.4 * mpx);
  double walk = 0.0;
  const int passes = tv3d_passes(n_inner);
  for (int i = 0, k = 0; i < passes; ++i) {
    const int T = tv3d_pass_steps(n_inner - k, passes - i);
    Tv3dSplit& s = split[T];
    if (s.rounds == 0) s = tv3d_split(g, T);
    walk += 2.0 + (double)s.rounds * (s.CY + 2 * T) * (i == 0 ? first_us : plane_us)[T];
    k += T;
  }
  return 1.03 * walk < two;
}

static hipError_t tv3d_pass(const ProxGeom& g, const Tv3dSplit& sp, int T, const float2* v, float2* const* p,
                            float2* const* po, float m0, const float* mom, float2* const* out,
                            float2* const* out_prev, float tau, float bound, hipStream_t s) {
  Tv3dArgs a{};
  a.Nz = g.Nz;
  a.Nx = g.Nx;
  a.Ny = g.Ny;
  a.ntz = sp.ntz;
  a.ntl = sp.ntl;
  a.nty = sp.nty;
  a.CY = sp.CY;
  const int64_t tiles = sp.cols * sp.nty;
  if (tiles > (int64_t)1 << 30) return hipErrorInvalidConfiguration;
  a.ntiles = (int)tiles;
  a.tau = tau;
  a.step = 1.0f / (12.0f * tau);
  a.bound = bound;
  a.m0 = m0;
  for (int t = 0; t < T; ++t) a.mom[t] = mom[t];
  a.v = v;
  a.cold = p[0] == nullptr;
  for (int c = 0; c < 3; ++c) {
    a.p[c] = a.cold ? v : p[c];   // a cold start loads (and ignores) something readable
    a.po[c] = po[c];
    a.out[c] = out[c];
    a.out_prev[c] = T > 1 ? out_prev[c] : nullptr;
  }
  const dim3 nb((a.ntiles + 7) & ~7), nt(TV3_WAVES * 64);
  const bool first = po[0] == nullptr;
  switch (T) {
    case 1:
      if (first) hipLaunchKernelGGL((tv3d_march_kernel<1, true>), nb, nt, 0, s, a);
      else hipLaunchKernelGGL((tv3d_march_kernel<1, false>), nb, nt, 0, s, a);
      break;
    case 2:
      if (first) hipLaunchKernelGGL((tv3d_march_kernel<2, true>), nb, nt, 0, s, a);
      else hipLaunchKernelGGL((tv3d_march_kernel<2, false>), nb, nt, 0, s, a);
      break;
    case 3:
      if (first) hipLaunchKernelGGL((tv3d_march_kernel<3, true>), nb, nt, 0, s, a);
      else hipLaunchKernelGGL((tv3d_march_kernel<3, false>), nb, nt, 0, s, a);
      break;
    default: return hipErrorInvalidValue;
  }
  return hipGetLastError();
}

// Inner steps of the 3-D path.  Runs of T steps (3 and 2) alternate between two
// pairs of duals, {last, previous} each: one pair holds p_out, the other is
// made of the scratch (work: four images, z and img_scratch: one each, z being
// written only after the steps; and scratch, three, which may be p_in: it is
// read by the first pass only, which does not write scratch).
static hipError_t tv3d_steps(const ProxGeom& g, const Tv3dSplit* split, int n_inner, const float* mom,
                             const float2* v, float2* z, const float2* p_in, float2* p_out, const Dual3& scratch,
                             float tau, float bound, float2* work, float2* img_scratch, hipStream_t s) {
  const int64_t n = (int64_t)g.B * g.Ny * g.Nx * g.Nz;
  auto packed = [&](const float2* p) {
    float2* q = const_cast<float2*>(p);
    return q ? Dual3{{q, q + n, q + 2 * n}} : Dual3{{nullptr, nullptr, nullptr}};
  };
  const Dual3 in = packed(p_in), out = packed(p_out), s1 = packed(work), s2{{work + 3 * n, z, img_scratch}},
              none = packed(nullptr);
  const int passes = tv3d_passes(n_inner);
  Dual3 last = in, prev = none;
  int k = 0;
  for (int i = 0; i < passes; ++i) {
    const int T = tv3d_pass_steps(n_inner - k, passes - i);
    const int left = passes - 1 - i;
    // where this pass leaves its last two duals: the pair with p_out when an even
    // number of passes is left (nothing follows the last one); scratch is in the
    // pair that the first pass does not write
    const bool outer = left % 2 == 0, scratch_with_out = passes % 2 == 0;
    const Dual3 o = outer ? out : s2;
    const Dual3 op = left == 0 ? none : outer == scratch_with_out ? scratch : s1;
    const hipError_t e = tv3d_pass(g, split[T], T, v, last.c, prev.c, k > 0 ? mom[k - 1] : 0.f, mom + k, o.c, op.c,
                                   tau, bound, s);
    if (e != hipSuccess) return e;
    prev = op;
    last = o;
    k += T;
  }
  return hipSuccess;
}

// p_in (nullable = zero) -> p_out; z = v + tau div p_out; partial (nullable:
// not computed) = TV(z).
hipError_t launch_prox_tv(const ProxGeom& g, int n_inner, const float* mom, const float2* v, float2* z,
                          const float2* p_in, float2* p_out, const Dual3& scratch, float tau, float bound,
                          double* partial, float2* work, float2* img_scratch, hipStream_t s) {
  if (tv_tiled(g, n_inner)) {
    Tv2dArgs a{};
    a.Nz = g.Nz;
    a.Nx = g.Nx;
    a.H = n_inner + 1;
    a.n_inner = n_inner;
    const Tv2dTiles t = tv2d_tiles(g, n_inner, partial != nullptr);
    a.CZ = t.CZ;
    a.CL = t.CL;
    a.ntz = t.ntz;
    a.ntl = t.ntl;
    a.n_total = (int64_t)g.B * g.Nx * g.Nz;
    a.tau = tau;
    a.step = 1.0f / (8.0f * tau);
    a.bound = bound;
    for (int k = 0; k < n_inner; ++k) a.mom[k] = mom[k];
    a.mom[n_inner] = 1.f;   // the last step leaves the plain dual in the kernel's P
    a.v = v;
    a.z = z;
    a.pin = p_in;
    a.pout = p_out;
    a.partial = partial;
    a.ntiles = a.ntz * a.ntl * g.B;
    const int nb = (a.ntiles + 7) & ~7;
    if (t.waves == TV_W1) tv2d_launch<TV_S1, TV_W1>(a, nb, bound, s);
    else tv2d_launch<TV_S2, TV_W2>(a, nb, bound, s);
    return hipGetLastError();
  }
  TvIdx d;
  d.Nz = g.Nz;
  d.Nx = g.Nx;
  d.Ny = (g.lateral_dims == 2) ? g.Ny : 1;
  d.nd = g.lateral_dims + 1;
  d.n = (int64_t)g.B * g.Ny * g.Nx * g.Nz;
  d.fast = d.n < (int64_t(1) << 32);
  d.fz = make_fastdiv((uint32_t)d.Nz);
  d.fx = make_fastdiv((uint32_t)d.Nx);
  d.fy = make_fastdiv((uint32_t)d.Ny);
  // batch items are independent: the y index wraps per item only for volumes;
  // for B-scans Ny = 1 and the x index never crosses a batch boundary because
  // coordinates are taken modulo each axis length.
  const int64_t np = d.n * d.nd;
  const int gb = grid_for(d.n, 256);
  Tv3dSplit split[TV3_MAX_T + 1] = {};
  if (g.lateral_dims == 1 || !tv3d_walks(g, n_inner, split)) {   // two kernels per step (B-scans: past the tile kernel's halo)
    float2* dd = work;
    float2* r = work + d.n;
    if (p_in) {
      hipLaunchKernelGGL(copy_kernel, dim3(grid_for(np, 256)), dim3(256), 0, s, p_in, p_out, np);
    } else {
      hipLaunchKernelGGL(zero_kernel, dim3(grid_for(np, 256)), dim3(256), 0, s, p_out, np);
    }
    hipLaunchKernelGGL(copy_kernel, dim3(grid_for(np, 256)), dim3(256), 0, s, p_out, r, np);
    const float step = 1.0f / (4.0f * d.nd * tau);
    for (int k = 0; k < n_inner; ++k) {
      hipLaunchKernelGGL(tv_div_kernel, dim3(gb), dim3(256), 0, s, d, v, r, tau, bound, dd);
      hipLaunchKernelGGL(tv_step_kernel, dim3(gb), dim3(256), 0, s, d, dd, r, p_out, step, mom[k]);
    }
  } else {
    const hipError_t e = tv3d_steps(g, split, n_inner, mom, v, z, p_in, p_out, scratch, tau, bound, work, img_scratch, s);
    if (e != hipSuccess) return e;
  }
  hipLaunchKernelGGL(tv_div_kernel, dim3(gb), dim3(256), 0, s, d, v, p_out, tau, bound, z);
  if (partial) hipLaunchKernelGGL(tv_value_kernel, dim3(gb), dim3(256), 0, s, d, z, partial);
  return hipGetLastError();
}
