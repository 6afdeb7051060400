// Dual-tree complex wavelet transform (Sec. 2.2; the DT-CWT of Selesnick,
// Baraniuk and Kingsbury) for B-scans, and its shrinkage step.
//
// Filters (designed on the host at first use, FP64, rounded once): Selesnick's
// common-factor construction of approximate Hilbert-transform pairs,
// h = F D and g = F D~, D the degree-L maximally flat allpass denominator for
// a half-sample delay (D~(z) = z^-L D(1/z)) and F = Q (1 + 1/z)^K with Q the
// minimum-phase spectral factor of the symmetric R that makes
// (z + 2 + 1/z)^K D(z) D(1/z) R(z) halfband.  First level: the 6-tap
// Daubechies filter (K = 3, L = 0) for tree a and the same one sample later
// for tree b; later levels: the 12-tap pair (K = 3, L = 3).
//
// Transform: four separable orthonormal 2-D DWTs (depth filters of tree a
// or b x lateral filters of tree a or b), periodic extension, both axes and
// all four trees of a level in one pass, bands in Mallat layout in one buffer
// per tree.  The detail bands of the four trees combine per element
// into the six oriented complex subbands (u1, v1) = (aa - bb, ab + ba)/sqrt2,
// (u2, v2) = (aa + bb, ab - ba)/sqrt2.  With the 1/2 scaling of the trees the
// transform W is a Parseval frame; the shrinkage step W^T soft_tau(W v) is
// computed on the unscaled trees as 1/4 sum_t T_t^T(C^T soft_{2 tau}(C T v)).
#include "oct_fft.h"

#include <cmath>
#include <complex>
#include <vector>

namespace {

constexpr int DT_MAXT = 16;

struct DtFilt {
  float h0[DT_MAXT], h1[DT_MAXT];
  int n;
};

// Periodic one-level filter banks along one axis of the top-left nx x nz
// sub-array of every image of the batch.  Analysis: lo[i] = sum_k h0[k]
// x[(2i + k) mod n], hi[i] likewise with h1, lo to the first half of the
// axis and hi to the second.  Synthesis is its transpose (the analysis is
// orthogonal): x[m] = sum over k with m - k even of h0[k] lo[i] + h1[k] hi[i],
// i = ((m - k) mod n) / 2.

__device__ __forceinline__ void fma2(float2& acc, float w, float2 x) {
  acc.x = fmaf(w, x.x, acc.x);
  acc.y = fmaf(w, x.y, acc.y);
}

__device__ __forceinline__ void afb_line(const DtFilt& f, const float2* __restrict__ src, int64_t stride, int n,
                                         int i, float2& lo, float2& hi) {
  lo = make_float2(0.f, 0.f);
  hi = make_float2(0.f, 0.f);
  int m = 2 * i;
  for (int k = 0; k < f.n; ++k) {
    const float2 x = src[(int64_t)m * stride];
    fma2(lo, f.h0[k], x);
    fma2(hi, f.h1[k], x);
    if (++m == n) m = 0;
  }
}

__device__ __forceinline__ float2 sfb_line(const DtFilt& f, const float2* __restrict__ src, int64_t stride, int n,
                                           int m) {
  const int h = n / 2;
  float2 x = make_float2(0.f, 0.f);
  for (int k = m & 1; k < f.n; k += 2) {
    int d = m - k;
    while (d < 0) d += n;
    const int i = d >> 1;
    fma2(x, f.h0[k], src[(int64_t)i * stride]);
    fma2(x, f.h1[k], src[(int64_t)(h + i) * stride]);
  }
  return x;
}

__device__ __forceinline__ float2 add2(float2 a, float2 b) { return make_float2(a.x + b.x, a.y + b.y); }
__device__ __forceinline__ float2 sub2(float2 a, float2 b) { return make_float2(a.x - b.x, a.y - b.y); }

// Combination of the four trees at one detail position into the two complex
// coefficients (u1, v1), (u2, v2); SHRINK shrinks both by tau2 and writes the
// trees back through the inverse combination, otherwise the moduli are added
// (scaled by 1/2 for the Parseval normalisation).
template <bool SHRINK>
__device__ __forceinline__ void dt_group(float2 (&w)[4], float tau2, double& acc) {
  const float r2 = 0.70710678118654752440f;
  float2 u1 = cscale(sub2(w[0], w[3]), r2), v1 = cscale(add2(w[1], w[2]), r2);
  float2 u2 = cscale(add2(w[0], w[3]), r2), v2 = cscale(sub2(w[1], w[2]), r2);
  const float m1 = sqrtf(u1.x * u1.x + u1.y * u1.y + v1.x * v1.x + v1.y * v1.y);
  const float m2 = sqrtf(u2.x * u2.x + u2.y * u2.y + v2.x * v2.x + v2.y * v2.y);
  if (!SHRINK) {
    acc += 0.5 * ((double)m1 + (double)m2);
    return;
  }
  const float s1 = m1 > tau2 ? 1.f - tau2 / m1 : 0.f;
  const float s2 = m2 > tau2 ? 1.f - tau2 / m2 : 0.f;
  u1 = cscale(u1, s1);
  v1 = cscale(v1, s1);
  u2 = cscale(u2, s2);
  v2 = cscale(v2, s2);
  w[0] = cscale(add2(u1, u2), r2);
  w[3] = cscale(sub2(u2, u1), r2);
  w[1] = cscale(add2(v1, v2), r2);
  w[2] = cscale(sub2(v1, v2), r2);
}

// Threads a register-window pass needs before it replaces the per-tap kernel
// (about four workgroups per CU): below that the walk along the axis leaves
// too few threads, and the per-tap kernel's rows fit the caches anyway.
constexpr int64_t DT_WINDOW_MIN_THREADS = (int64_t)1 << 18;

// One level of a B-scan's four trees (tree 2 d + l: depth filter d, lateral
// filter l; 0 = a, 1 = b).  nx x nz is the sub-array at the top-left of every
// item that the level splits (analysis) or rebuilds (synthesis).
struct DtLevel {
  int B, NX, NZ, nx, nz;
  const float2* src;   // tree t at src + t * sstride
  float2* dst;         // tree t at dst + t * dstride
  int64_t sstride, dstride;
  float f[2][2][12];   // [filter a, b][h0, h1][tap]
};

// One analysis level, both axes and all four trees in one pass.  Four separate
// lateral and depth passes moved every tree through memory twice per level with
// one load per tap.  A workgroup owns DZ depth x P G lateral outputs of every
// band: each thread walks 2 P + NT - 2 rows of one depth column (all loads
// independent, coalesced along depth; every row of a column is loaded once per
// P outputs) and leaves the lateral bands in LDS; the depth filters then run
// along LDS rows by 16-byte reads, and one thread holds all four trees of a
// position, as the shrinkage of the details needs.  Lateral-low depth-low
// outputs are the next level's low band and are written as they are; every
// other output is a detail coefficient, combined across the trees and shrunk
// (SHRINK, then written) or summed into an FP64 block partial (value pass: only
// the low band is written).  NS = 1: the first level, where the trees share one
// source; NS = 4: a source per tree.  Sources and destinations are different
// buffers (workgroups read their neighbours' rows).
// Bound: 16 MB in and 66 MB out at the first level of a 2048 x 1000 B-scan
// (17 us at the copy rate); measured 18.1 us there and 11.5 + 7.4 at the next
// two levels, 37 in all, where the separate depth and lateral passes took 95.
template <bool SHRINK, int NT, int NS, int DZ, int P, int G, int THREADS>
__global__ void __launch_bounds__(THREADS) dt_analysis_kernel(DtLevel a, float tau2, double* partial) {
  constexpr int RX = P * G, PW = 2 * DZ + NT - 2, NA = NS == 1 ? 2 : 4;
  static_assert(PW % 2 == 0, "16-byte LDS rows");
  __shared__ __align__(16) float2 band[NA][2][RX][PW];
  const int h = a.nx / 2, hz = a.nz / 2;
  const int tz = (hz + DZ - 1) / DZ, tx = (h + RX - 1) / RX;
  const int64_t tiles = (int64_t)a.B * tx * tz;
  double acc = 0.0;
  for (int64_t tile = blockIdx.x; tile < tiles; tile += gridDim.x) {
    const int i0 = (int)(tile % tz) * DZ, r0 = (int)(tile / tz % tx) * RX;
    const int64_t item = tile / tz / tx * a.NX * a.NZ;
    if (tile != blockIdx.x) __syncthreads();
    for (int e = threadIdx.x; e < NS * G * PW; e += THREADS) {
      const int c = e % PW, g = e / PW % G, t = e / PW / G;
      const int r = r0 + g * P;
      if (r >= h) continue;
      const float2* p = a.src + t * a.sstride + item + (int64_t)(2 * r) * a.NZ + (2 * i0 + c) % a.nz;
      float2 x[2 * P + NT - 2];
      int m = 2 * r;
#pragma unroll
      for (int u = 0; u < 2 * P + NT - 2; ++u) {
        x[u] = *p;
        p += a.NZ;
        if (++m == a.nx) {
          m = 0;
          p -= (int64_t)a.nx * a.NZ;
        }
      }
#pragma unroll
      for (int l = 0; l < (NS == 1 ? 2 : 1); ++l) {
        const bool fb = NS == 1 ? l == 1 : (t & 1) == 1;
        float2 lo[P], hi[P];
#pragma unroll
        for (int o = 0; o < P; ++o) lo[o] = hi[o] = make_float2(0.f, 0.f);
#pragma unroll
        for (int k = 0; k < NT; ++k) {
          const float w0 = fb ? a.f[1][0][k] : a.f[0][0][k];
          const float w1 = fb ? a.f[1][1][k] : a.f[0][1][k];
#pragma unroll
          for (int o = 0; o < P; ++o) {
            fma2(lo[o], w0, x[2 * o + k]);
            fma2(hi[o], w1, x[2 * o + k]);
          }
        }
        const int arr = NS == 1 ? l : t;
#pragma unroll
        for (int o = 0; o < P; ++o) {
          band[arr][0][g * P + o][c] = lo[o];
          band[arr][1][g * P + o][c] = hi[o];
        }
      }
    }
    __syncthreads();
    for (int e = threadIdx.x; e < RX * DZ; e += THREADS) {
      const int c = e % DZ, row = e / DZ;
      const int i = i0 + c, r = r0 + row;
      if (i >= hz || r >= h) continue;
      float2 ll[4], lh[4], hl[4], hh[4];   // [lateral band][depth band]
#pragma unroll
      for (int q = 0; q < NA; ++q) {
#pragma unroll
        for (int lat = 0; lat < 2; ++lat) {
          float2 x[NT];
          const float4* row4 = reinterpret_cast<const float4*>(&band[q][lat][row][2 * c]);
#pragma unroll
          for (int k = 0; k < NT / 2; ++k) {
            const float4 v = row4[k];
            x[2 * k] = make_float2(v.x, v.y);
            x[2 * k + 1] = make_float2(v.z, v.w);
          }
#pragma unroll
          for (int s = 0; s < (NS == 1 ? 2 : 1); ++s) {
            const int t = NS == 1 ? 2 * s + q : q, d = t >> 1;
            float2 lo = make_float2(0.f, 0.f), hi = make_float2(0.f, 0.f);
#pragma unroll
            for (int k = 0; k < NT; ++k) {
              fma2(lo, a.f[d][0][k], x[k]);
              fma2(hi, a.f[d][1][k], x[k]);
            }
            // one LDS row's taps at a time: with all in flight the registers leave one workgroup per CU
            asm volatile("" : "+v"(lo.x), "+v"(lo.y), "+v"(hi.x), "+v"(hi.y)::"memory");
            if (lat == 0) {
              ll[t] = lo;
              lh[t] = hi;
            } else {
              hl[t] = lo;
              hh[t] = hi;
            }
          }
        }
      }
      dt_group<SHRINK>(lh, tau2, acc);
      dt_group<SHRINK>(hl, tau2, acc);
      dt_group<SHRINK>(hh, tau2, acc);
      float2* olo = a.dst + item + (int64_t)r * a.NZ + i;
      float2* ohi = olo + (int64_t)h * a.NZ;
#pragma unroll
      for (int t = 0; t < 4; ++t) {
        olo[t * a.dstride] = ll[t];
        if (SHRINK) {
          olo[t * a.dstride + hz] = lh[t];
          ohi[t * a.dstride] = hl[t];
          ohi[t * a.dstride + hz] = hh[t];
        }
      }
    }
  }
  if (!SHRINK) {
    __shared__ double sh[THREADS / 64];
#pragma unroll
    for (int o = 32; o > 0; o >>= 1) acc += __shfl_xor(acc, o);
    const int lane = threadIdx.x & 63, w = threadIdx.x >> 6;
    if (lane == 0) sh[w] = acc;
    __syncthreads();
    if (threadIdx.x == 0) {
      double s = 0.0;
      for (int k = 0; k < THREADS / 64; ++k) s += sh[k];
      partial[blockIdx.x] = s;
    }
  }
}

// One synthesis level (the transpose of the analysis), both axes in one pass.
// A workgroup owns 2 DZ depth x 2 P G lateral outputs.  Outputs 2p and 2p + 1
// read the same NT / 2 rows p - NT / 2 + 1 .. p of each band, so a thread takes
// P row pairs of one depth column of one depth band (P + NT / 2 - 1 rows of
// both lateral bands, all loads independent) and leaves the laterally
// synthesised column in LDS; the depth synthesis reads it there, each thread
// with the taps of its own parity, and writes along depth.  ND = 2: the first
// level, the four trees summed into dst (both lateral trees of a depth filter
// before LDS) and scaled; ND = 1: one tree per blockIdx.y.  Sources and
// destinations are different buffers.
// Bound: 66 MB in and 16 MB out at the first level of a 2048 x 1000 B-scan
// (17 us at the copy rate); measured 21.7 us there and 16.8 for the two levels
// below, 38 in all, where the separate lateral and depth passes took 124.
template <int NT, int ND, int DZ, int P, int G, int THREADS>
__global__ void __launch_bounds__(THREADS) dt_synthesis_kernel(DtLevel a, float scale) {
  constexpr int W = NT / 2, RX = P * G, CW = DZ + W - 1;
  static_assert(THREADS % 2 == 0, "a thread keeps its parity");
  __shared__ float2 mid[ND][2 * RX][2 * CW];
  const int h = a.nx / 2, hz = a.nz / 2;
  const int tz = (hz + DZ - 1) / DZ, tx = (h + RX - 1) / RX;
  const int64_t tiles = (int64_t)a.B * tx * tz;
  const int tree = blockIdx.y;
  const int par = threadIdx.x & 1;
  for (int64_t tile = blockIdx.x; tile < tiles; tile += gridDim.x) {
    const int i0 = (int)(tile % tz) * DZ, r0 = (int)(tile / tz % tx) * RX;
    const int64_t item = tile / tz / tx * a.NX * a.NZ;
    if (tile != blockIdx.x) __syncthreads();
    for (int e = threadIdx.x; e < ND * G * 2 * CW; e += THREADS) {
      const int c = e % (2 * CW), g = e / (2 * CW) % G, d = e / (2 * CW) / G;
      const int p0 = r0 + g * P;
      if (p0 >= h) continue;
      int i = (i0 - (W - 1) + (c >= CW ? c - CW : c)) % hz;
      if (i < 0) i += hz;
      int m = (p0 - (W - 1)) % h;
      if (m < 0) m += h;
      const int64_t off = item + (int64_t)m * a.NZ + (c >= CW ? hz + i : i);
      float2 x[2 * P];
#pragma unroll
      for (int o = 0; o < 2 * P; ++o) x[o] = make_float2(0.f, 0.f);
#pragma unroll
      for (int l = 0; l < ND; ++l) {
        const int t = ND == 2 ? 2 * d + l : tree;
        const float* f0 = ND == 2 ? a.f[l][0] : a.f[tree & 1][0];
        const float* f1 = ND == 2 ? a.f[l][1] : a.f[tree & 1][1];
        const float2* p = a.src + t * a.sstride + off;
        float2 lo[P + W - 1], hi[P + W - 1];
        int mm = m;
#pragma unroll
        for (int u = 0; u < P + W - 1; ++u) {
          lo[u] = *p;
          hi[u] = p[(int64_t)h * a.NZ];
          p += a.NZ;
          if (++mm == h) {
            mm = 0;
            p -= (int64_t)h * a.NZ;
          }
        }
#pragma unroll
        for (int k = 0; k < NT; ++k) {
#pragma unroll
          for (int o = 0; o < P; ++o) {
            fma2(x[2 * o + (k & 1)], f0[k], lo[o + W - 1 - (k >> 1)]);
            fma2(x[2 * o + (k & 1)], f1[k], hi[o + W - 1 - (k >> 1)]);
          }
        }
      }
#pragma unroll
      for (int o = 0; o < 2 * P; ++o) mid[d][2 * g * P + o][c] = x[o];
    }
    __syncthreads();
    float w0[ND][W], w1[ND][W];
#pragma unroll
    for (int d = 0; d < ND; ++d) {
      const int fd = ND == 2 ? d : tree >> 1;
#pragma unroll
      for (int k = 0; k < W; ++k) {
        w0[d][k] = par ? a.f[fd][0][2 * k + 1] : a.f[fd][0][2 * k];
        w1[d][k] = par ? a.f[fd][1][2 * k + 1] : a.f[fd][1][2 * k];
      }
    }
    for (int e = threadIdx.x; e < 2 * RX * 2 * DZ; e += THREADS) {
      const int c = e % (2 * DZ), row = e / (2 * DZ);
      const int n = 2 * i0 + c, r = 2 * r0 + row;
      if (n >= a.nz || r >= a.nx) continue;
      float2 v = make_float2(0.f, 0.f);
#pragma unroll
      for (int d = 0; d < ND; ++d) {
        const float2* q = &mid[d][row][(c >> 1) + W - 1];
        float2 x = make_float2(0.f, 0.f);
#pragma unroll
        for (int k = 0; k < W; ++k) {
          fma2(x, w0[d][k], q[-k]);
          fma2(x, w1[d][k], q[CW - k]);
        }
        v = d == 0 ? x : make_float2(v.x + x.x, v.y + x.y);
      }
      a.dst[tree * a.dstride + item + (int64_t)r * a.NZ + n] = make_float2(scale * v.x, scale * v.y);
    }
  }
}

int dt_grid(int64_t n) {
  int64_t b = (n + 255) / 256;
  if (b > 4096) b = 4096;
  return (int)(b < 1 ? 1 : b);
}

// ---------------------------------------------------------------------------
// Host filter design (FP64)
// ---------------------------------------------------------------------------
std::vector<double> conv(const std::vector<double>& a, const std::vector<double>& b) {
  std::vector<double> o(a.size() + b.size() - 1, 0.0);
  for (size_t i = 0; i < a.size(); ++i)
    for (size_t j = 0; j < b.size(); ++j) o[i + j] += a[i] * b[j];
  return o;
}

double binom(int n, int k) {
  double v = 1.0;
  for (int i = 1; i <= k; ++i) v = v * (double)(n - k + i) / (double)i;
  return v;
}

// Gaussian elimination with partial pivoting (n x n, row-major), in place.
bool solve(std::vector<double>& A, std::vector<double>& b, int n) {
  for (int c = 0; c < n; ++c) {
    int p = c;
    for (int r = c + 1; r < n; ++r)
      if (std::fabs(A[r * n + c]) > std::fabs(A[p * n + c])) p = r;
    if (std::fabs(A[p * n + c]) < 1e-300) return false;
    if (p != c) {
      for (int k = 0; k < n; ++k) std::swap(A[p * n + k], A[c * n + k]);
      std::swap(b[p], b[c]);
    }
    for (int r = c + 1; r < n; ++r) {
      const double f = A[r * n + c] / A[c * n + c];
      for (int k = c; k < n; ++k) A[r * n + k] -= f * A[c * n + k];
      b[r] -= f * b[c];
    }
  }
  for (int c = n - 1; c >= 0; --c) {
    double s = b[c];
    for (int k = c + 1; k < n; ++k) s -= A[c * n + k] * b[k];
    b[c] = s / A[c * n + c];
  }
  return true;
}

// Roots of sum_i p[i] z^(deg - i) (p[0] != 0) by the Weierstrass (Durand-Kerner)
// iteration.
std::vector<std::complex<double>> roots(const std::vector<double>& p) {
  const int deg = (int)p.size() - 1;
  std::vector<std::complex<double>> z(deg);
  const std::complex<double> seed(0.4, 0.9);
  for (int i = 0; i < deg; ++i) z[i] = std::pow(seed, i);
  for (int it = 0; it < 2000; ++it) {
    double move = 0.0;
    for (int i = 0; i < deg; ++i) {
      std::complex<double> num = p[0];
      for (int k = 1; k <= deg; ++k) num = num * z[i] + p[k];
      std::complex<double> den = p[0];
      for (int j = 0; j < deg; ++j)
        if (j != i) den *= (z[i] - z[j]);
      const std::complex<double> d = num / den;
      z[i] -= d;
      move = std::max(move, std::abs(d));
    }
    if (move < 1e-15) break;
  }
  return z;
}

// Lowpass pair (h, g) of the common-factor design with K zeros at z = -1 and a
// degree-L half-sample allpass (L = 0: Daubechies, h = g).
void design_pair(int K, int L, std::vector<double>& h, std::vector<double>& g) {
  std::vector<double> d(L + 1);
  for (int n = 0; n <= L; ++n) {
    double v = (n & 1) ? -binom(L, n) : binom(L, n);
    for (int k = 0; k < n; ++k) v *= (0.5 - L + k) / (1.5 + k);
    d[n] = v;
  }
  std::vector<double> dr(d.rbegin(), d.rend());
  std::vector<double> q0 = conv(d, dr);
  for (int k = 0; k < K; ++k) q0 = conv(q0, {1.0, 2.0, 1.0});
  const int M = K + L - 1, nP = K + L + M;
  const int neq = (nP + 1) / 2;           // = M + 1
  std::vector<double> A(neq * neq), rhs(neq, 0.0);
  rhs[0] = 1.0;
  for (int i = 0; i <= M; ++i) {
    std::vector<double> r(2 * M + 1, 0.0);
    r[M + i] = 1.0;
    r[M - i] = 1.0;
    const std::vector<double> col = conv(q0, r);    // centre index nP
    for (int e = 0; e < neq; ++e) A[e * neq + i] = col[nP + 2 * e];
  }
  solve(A, rhs, neq);
  std::vector<double> f = {1.0};
  if (M > 0) {
    std::vector<double> R(2 * M + 1);
    R[M] = rhs[0];
    for (int i = 1; i <= M; ++i) R[M + i] = R[M - i] = rhs[i];
    // minimum-phase factor: the monic polynomial of the roots inside the unit circle
    std::vector<std::complex<double>> poly = {1.0};
    for (const auto& z : roots(R))
      if (std::abs(z) < 1.0) {
        std::vector<std::complex<double>> nx(poly.size() + 1, 0.0);
        for (size_t k = 0; k < poly.size(); ++k) {
          nx[k] += poly[k];
          nx[k + 1] -= poly[k] * z;
        }
        poly = nx;
      }
    f.assign(poly.size(), 0.0);
    for (size_t k = 0; k < poly.size(); ++k) f[k] = poly[k].real();
  }
  for (int k = 0; k < K; ++k) f = conv(f, {1.0, 1.0});
  h = conv(f, d);
  g = conv(f, dr);
  double s = 0.0;
  for (double v : h) s += v;
  const double sc = std::sqrt(2.0) / s;
  for (double& v : h) v *= sc;
  for (double& v : g) v *= sc;
}

DtFilt make_filt(const std::vector<double>& h) {
  DtFilt f{};
  f.n = (int)h.size();
  for (int k = 0; k < f.n; ++k) {
    f.h0[k] = (float)h[k];
    const double hk = h[f.n - 1 - k];
    f.h1[k] = (float)((k & 1) ? -hk : hk);
  }
  return f;
}

struct DtFilters {
  DtFilt first[2], later[2];
};

DtFilters design_filters() {
  DtFilters F;
  std::vector<double> d1, d1g, ha, hb;
  design_pair(3, 0, d1, d1g);
  std::vector<double> fa(d1), fb(1, 0.0);
  fa.push_back(0.0);
  fa.push_back(0.0);
  fb.insert(fb.end(), d1.begin(), d1.end());
  fb.push_back(0.0);
  design_pair(3, 3, ha, hb);
  F.first[0] = make_filt(fa);
  F.first[1] = make_filt(fb);
  F.later[0] = make_filt(ha);
  F.later[1] = make_filt(hb);
  return F;
}

// Designed once per process (the initialisation of a function-local static
// is thread safe: plans on several host threads may ask at once).
const DtFilters& filters() {
  static const DtFilters F = design_filters();
  return F;
}

int dt_grid_y(int64_t n, int jobs) {
  int64_t b = (n + 255) / 256;
  const int64_t cap = 4096 / jobs;
  if (b > cap) b = cap;
  return (int)(b < 1 ? 1 : b);
}

// Tile shapes of a B-scan's levels: depth outputs per band, lateral outputs
// (or output pairs) per thread, threads' groups along the lateral axis, threads.
// Enough threads that the columns of a tile take one turn (NS G (2 DZ + NT - 2)
// and 2 ND G (DZ + NT / 2 - 1)) and workgroups small enough to overlap one's
// loads with another's filters.  Measured at 2048 x 1000 (us): first analysis
// 18.1 (G = 4 18.7, DZ = 64 18.6, P = 8 20.6, 320 threads at G = 4 20.5);
// levels 2 and 3 of the analysis 11.5 + 7.4 (P = 4 13.4 + 6.6, G = 2 13.0 +
// 7.8); first synthesis 21.7 (DZ = 32 with G = 4 22.2, G = 2 23.6, P = 8 30.5);
// later synthesis 10.5 + 6.3 (G = 2 12.0 + 5.6, P = 8 12.2 + 6.7).
constexpr int DTA1_DZ = 32, DTA1_P = 4, DTA1_G = 2, DTA1_T = 256;
constexpr int DTA2_DZ = 32, DTA2_P = 8, DTA2_G = 1, DTA2_T = 320;
constexpr int DTS1_DZ = 64, DTS1_P = 4, DTS1_G = 2, DTS1_T = 256;
constexpr int DTS2_DZ = 32, DTS2_P = 4, DTS2_G = 3, DTS2_T = 256;
constexpr int DT_N1 = 8, DT_N2 = 12;   // taps of the first level's and the later levels' filters

DtLevel dt_level(const ProxGeom& pg, int lev) {
  const DtFilters& F = filters();
  DtLevel a{};
  a.B = pg.B;
  a.NX = pg.Nx;
  a.NZ = pg.Nz;
  a.nx = pg.Nx >> lev;
  a.nz = pg.Nz >> lev;
  for (int t = 0; t < 2; ++t) {
    const DtFilt& f = lev == 0 ? F.first[t] : F.later[t];
    for (int k = 0; k < f.n; ++k) {
      a.f[t][0][k] = f.h0[k];
      a.f[t][1][k] = f.h1[k];
    }
  }
  return a;
}

unsigned dt_tiles(const DtLevel& a, int dz, int rx, int64_t cap) {
  const int64_t n = (int64_t)a.B * ((a.nz / 2 + dz - 1) / dz) * ((a.nx / 2 + rx - 1) / rx);
  return (unsigned)(n < cap ? n : cap);
}

unsigned dt_analysis_grid(const DtLevel& a, int lev) {
  return lev == 0 ? dt_tiles(a, DTA1_DZ, DTA1_P * DTA1_G, 4096) : dt_tiles(a, DTA2_DZ, DTA2_P * DTA2_G, 4096);
}

// Level lev's bands live in the first four images of the workspace (lev even)
// or in the last four (odd): a level reads the low bands of the one before from
// the other half, so no workgroup overwrites what a neighbour still reads.
float2* dt_bands(const ProxGeom& pg, float2* work, int lev) {
  return work + (lev & 1) * 4 * ((int64_t)pg.B * pg.Nx * pg.Nz);
}

template <bool SHRINK>
void dt_analysis_level(const DtLevel& a, int lev, float tau2, double* partial, hipStream_t s) {
  const dim3 grid(dt_analysis_grid(a, lev));
  if (lev == 0)
    hipLaunchKernelGGL((dt_analysis_kernel<SHRINK, DT_N1, 1, DTA1_DZ, DTA1_P, DTA1_G, DTA1_T>), grid, dim3(DTA1_T), 0,
                       s, a, tau2, partial);
  else
    hipLaunchKernelGGL((dt_analysis_kernel<SHRINK, DT_N2, 4, DTA2_DZ, DTA2_P, DTA2_G, DTA2_T>), grid, dim3(DTA2_T), 0,
                       s, a, tau2, partial);
}

// Analysis of all trees, level by level.  mode 0: the detail bands shrunk by
// tau2 on the way; mode 1: the value pass (block partials of sum |W x| into
// partial, nothing but the low bands written).
hipError_t dt_analysis(const ProxGeom& pg, int levels, const float2* v, float2* work, int mode, float tau2,
                       double* partial, hipStream_t s) {
  const int64_t n = (int64_t)pg.B * pg.Nx * pg.Nz;
  for (int lev = 0; lev < levels; ++lev) {
    DtLevel a = dt_level(pg, lev);
    a.src = lev == 0 ? v : dt_bands(pg, work, lev - 1);
    a.sstride = lev == 0 ? 0 : n;
    a.dst = dt_bands(pg, work, lev);
    a.dstride = n;
    if (mode == 0) {
      dt_analysis_level<true>(a, lev, tau2, nullptr, s);
    } else {
      dt_analysis_level<false>(a, lev, 0.f, partial, s);
      partial += dt_analysis_grid(a, lev);
    }
  }
  return hipGetLastError();
}

// Synthesis, coarsest level first; the first level sums the trees into z.
hipError_t dt_synthesis(const ProxGeom& pg, int levels, float2* z, float2* work, hipStream_t s) {
  const int64_t n = (int64_t)pg.B * pg.Nx * pg.Nz;
  for (int lev = levels - 1; lev >= 0; --lev) {
    DtLevel a = dt_level(pg, lev);
    a.src = dt_bands(pg, work, lev);
    a.sstride = n;
    if (lev == 0) {
      a.dst = z;
      hipLaunchKernelGGL((dt_synthesis_kernel<DT_N1, 2, DTS1_DZ, DTS1_P, DTS1_G, DTS1_T>),
                         dim3(dt_tiles(a, DTS1_DZ, DTS1_P * DTS1_G, 4096)), dim3(DTS1_T), 0, s, a, 0.25f);
    } else {
      a.dst = dt_bands(pg, work, lev - 1);
      a.dstride = n;
      hipLaunchKernelGGL((dt_synthesis_kernel<DT_N2, 1, DTS2_DZ, DTS2_P, DTS2_G, DTS2_T>),
                         dim3(dt_tiles(a, DTS2_DZ, DTS2_P * DTS2_G, 1024), 4), dim3(DTS2_T), 0, s, a, 1.f);
    }
  }
  return hipGetLastError();
}

// ---------------------------------------------------------------------------
// Volumes: eight trees (depth, x, y filter trees), a pass per axis and level.
// ---------------------------------------------------------------------------
struct Dt3Geom {
  int B, NY, NX, NZ;  // image [B][NY][NX][NZ]
  int ny, nx, nz;     // current sub-array at the corner of every item
};

struct DtJobs8 {
  const float2* src[8];
  float2* dst[8];
  DtFilt f[8];
  float scale;
};

// Orthogonal combination of the eight tree values (tree index 4 tz + 2 tx +
// ty, a = 0, b = 1) of one detail coefficient into the real and imaginary
// parts of four complex coefficients (rows u0, v0, ..., u3, v3): the 3-D
// complex wavelet is the product over the axes of (tree a + j tree b), with
// the x and y factors optionally conjugated (signs sx, sy = ++, +-, -+, --):
// u = (aaa - sx sy abb - sx bba - sy bab)/2, v = (sx aba + sy aab + baa - sx sy bbb)/2.
__device__ __forceinline__ float dt3_c(int row, int t) {
  const int k = row >> 1;
  const float sx = (k & 2) ? -1.f : 1.f, sy = (k & 1) ? -1.f : 1.f;
  if ((row & 1) == 0) {
    switch (t) {
      case 0: return 0.5f;
      case 3: return -0.5f * sx * sy;
      case 6: return -0.5f * sx;
      case 5: return -0.5f * sy;
      default: return 0.f;
    }
  }
  switch (t) {
    case 2: return 0.5f * sx;
    case 1: return 0.5f * sy;
    case 4: return 0.5f;
    case 7: return -0.5f * sx * sy;
    default: return 0.f;
  }
}

template <bool SHRINK>
__device__ __forceinline__ void dt3_group(float2 (&w)[8], float tau2, double& acc) {
  float2 c[8];
#pragma unroll
  for (int r = 0; r < 8; ++r) {
    c[r] = make_float2(0.f, 0.f);
#pragma unroll
    for (int t = 0; t < 8; ++t) fma2(c[r], dt3_c(r, t), w[t]);
  }
#pragma unroll
  for (int k = 0; k < 4; ++k) {
    const float2 u = c[2 * k], v = c[2 * k + 1];
    const float m = sqrtf(u.x * u.x + u.y * u.y + v.x * v.x + v.y * v.y);
    if (!SHRINK) {
      acc += 0.35355339059327376220 * (double)m;   // 2^(-3/2): the trees' Parseval scale
    } else {
      const float sc = m > tau2 ? 1.f - tau2 / m : 0.f;
      c[2 * k] = cscale(u, sc);
      c[2 * k + 1] = cscale(v, sc);
    }
  }
  if (SHRINK) {
#pragma unroll
    for (int t = 0; t < 8; ++t) {
      w[t] = make_float2(0.f, 0.f);
#pragma unroll
      for (int r = 0; r < 8; ++r) fma2(w[t], dt3_c(r, t), c[r]);
    }
  }
}

__device__ __forceinline__ int64_t dt3_off(const Dt3Geom& g, int b, int y, int x, int n) {
  return (((int64_t)b * g.NY + y) * g.NX + x) * g.NZ + n;
}

// Analysis along one axis (0 depth, 1 x, 2 y) of the corner sub-array; the
// depth index runs fastest for the lateral axes (coalesced).
template <int AXIS>
__global__ void afb3_kernel(Dt3Geom g, DtJobs8 J) {
  const int j = blockIdx.y;
  const int len = AXIS == 0 ? g.nz : AXIS == 1 ? g.nx : g.ny;
  const int h = len / 2;
  const int64_t stride = AXIS == 0 ? 1 : AXIS == 1 ? (int64_t)g.NZ : (int64_t)g.NX * g.NZ;
  const int a0 = AXIS == 0 ? h : g.nz;                 // fastest index range
  const int a1 = AXIS == 1 ? h : g.nx;
  const int a2 = AXIS == 2 ? h : g.ny;
  const int64_t total = (int64_t)g.B * a2 * a1 * a0;
  for (int64_t t = blockIdx.x * (int64_t)blockDim.x + threadIdx.x; t < total; t += (int64_t)gridDim.x * blockDim.x) {
    const int i0 = (int)(t % a0);
    int64_t r = t / a0;
    const int i1 = (int)(r % a1);
    r /= a1;
    const int i2 = (int)(r % a2);
    const int b = (int)(r / a2);
    const int n = AXIS == 0 ? 0 : i0, x = AXIS == 1 ? 0 : i1, y = AXIS == 2 ? 0 : i2;
    const int i = AXIS == 0 ? i0 : AXIS == 1 ? i1 : i2;
    const int64_t base = dt3_off(g, b, y, x, n);
    float2 lo, hi;
    afb_line(J.f[j], J.src[j] + base, stride, len, i, lo, hi);
    J.dst[j][base + (int64_t)i * stride] = lo;
    J.dst[j][base + (int64_t)(h + i) * stride] = hi;
  }
}

// Synthesis along one axis; ACC sums job pairs (2y, 2y + 1) into dst[2y].
template <int AXIS, bool ACC>
__global__ void sfb3_kernel(Dt3Geom g, DtJobs8 J) {
  const int j = blockIdx.y * (ACC ? 2 : 1);
  const int len = AXIS == 0 ? g.nz : AXIS == 1 ? g.nx : g.ny;
  const int64_t stride = AXIS == 0 ? 1 : AXIS == 1 ? (int64_t)g.NZ : (int64_t)g.NX * g.NZ;
  const int64_t total = (int64_t)g.B * g.ny * g.nx * g.nz;
  for (int64_t t = blockIdx.x * (int64_t)blockDim.x + threadIdx.x; t < total; t += (int64_t)gridDim.x * blockDim.x) {
    const int n = (int)(t % g.nz);
    int64_t r = t / g.nz;
    const int x = (int)(r % g.nx);
    r /= g.nx;
    const int y = (int)(r % g.ny);
    const int b = (int)(r / g.ny);
    const int m = AXIS == 0 ? n : AXIS == 1 ? x : y;
    const int64_t base = dt3_off(g, b, AXIS == 2 ? 0 : y, AXIS == 1 ? 0 : x, AXIS == 0 ? 0 : n);
    float2 v = sfb_line(J.f[j], J.src[j] + base, stride, len, m);
    if (ACC) {
      const float2 w = sfb_line(J.f[j + 1], J.src[j + 1] + base, stride, len, m);
      v = make_float2(v.x + w.x, v.y + w.y);
    }
    J.dst[j][base + (int64_t)m * stride] = make_float2(J.scale * v.x, J.scale * v.y);
  }
}

// Lateral synthesis of the volume along x (AXIS 1) or y (AXIS 2) with a
// sliding register window.  Per output, sfb3_kernel fetches one input row per
// tap; rows 16 KB (x) or n_x n_z samples (y) apart are not held by the caches
// between neighbouring outputs, so each input came from memory about once per
// tap.  Outputs 2p and 2p + 1 read the same NT/2 rows i = p - NT/2 + 1 .. p of
// each band, so a thread that walks RP output pairs along the axis (one depth
// lane, one position of the other lateral axis) loads every row once, plus
// NT/2 - 1 rows at the start of its run, with no LDS and no barrier.  Window
// slots are fixed at compile time (the walk is unrolled).  Taps are applied
// in sfb_line's order and the per-tree sums added as in sfb3_kernel: the same
// result bit for bit.
template <int AXIS, bool ACC, int NT>
__global__ void __launch_bounds__(256) sfb3_window(Dt3Geom g, DtJobs8 J) {
  static_assert(AXIS == 1 || AXIS == 2, "lateral axes only");
  constexpr int W = NT / 2, RP = 16;
  constexpr int NS = ACC ? 2 : 1;
  const int j = blockIdx.y * NS;
  const int len = AXIS == 1 ? g.nx : g.ny, h = len / 2;
  const int others = AXIS == 1 ? g.ny : g.nx;
  const int runs = (h + RP - 1) / RP;
  const int64_t stride = AXIS == 1 ? (int64_t)g.NZ : (int64_t)g.NX * g.NZ;
  const int64_t total = (int64_t)g.B * others * runs * g.nz;
  for (int64_t t = blockIdx.x * (int64_t)blockDim.x + threadIdx.x; t < total; t += (int64_t)gridDim.x * blockDim.x) {
    const int n = (int)(t % g.nz);
    int64_t r = t / g.nz;
    const int run = (int)(r % runs);
    r /= runs;
    const int other = (int)(r % others);
    const int b = (int)(r / others);
    const int64_t item = (AXIS == 1 ? (((int64_t)b * g.NY + other) * g.NX) * g.NZ
                                    : ((int64_t)b * g.NY * g.NX + other) * g.NZ) + n;
    const int p0 = run * RP;
    // slot u % W holds band row p0 - W + 1 + u (mod h)
    float2 lo[NS][W], hi[NS][W];
#pragma unroll
    for (int u = 0; u < W - 1; ++u) {
      int i = (p0 - W + 1 + u) % h;
      if (i < 0) i += h;
#pragma unroll
      for (int q = 0; q < NS; ++q) {
        lo[q][u % W] = J.src[j + q][item + (int64_t)i * stride];
        hi[q][u % W] = J.src[j + q][item + (int64_t)(h + i) * stride];
      }
    }
#pragma unroll
    for (int sp = 0; sp < RP; ++sp) {
      const int p = p0 + sp;
      if (p < h) {
#pragma unroll
        for (int q = 0; q < NS; ++q) {
          lo[q][(W - 1 + sp) % W] = J.src[j + q][item + (int64_t)p * stride];
          hi[q][(W - 1 + sp) % W] = J.src[j + q][item + (int64_t)(h + p) * stride];
        }
#pragma unroll
        for (int odd = 0; odd < 2; ++odd) {
          float2 v = make_float2(0.f, 0.f);
#pragma unroll
          for (int q = 0; q < NS; ++q) {
            const DtFilt& f = J.f[j + q];
            float2 x = make_float2(0.f, 0.f);
#pragma unroll
            for (int k = odd; k < NT; k += 2) {
              const int slot = (W - 1 + sp - (k >> 1)) % W;
              fma2(x, f.h0[k], lo[q][slot]);
              fma2(x, f.h1[k], hi[q][slot]);
            }
            v = q == 0 ? x : make_float2(v.x + x.x, v.y + x.y);
          }
          J.dst[j][item + (int64_t)(2 * p + odd) * stride] = make_float2(J.scale * v.x, J.scale * v.y);
        }
      }
    }
  }
}

// y analysis of all eight trees in one thread with the level's detail bands
// combined and shrunk (or summed) on the spot, as in dt_analysis_kernel.
template <bool SHRINK>
__global__ void afb3_y8_kernel(Dt3Geom g, DtJobs8 J, float tau2, double* partial) {
  __shared__ double sh[16];
  const int h = g.ny / 2, hx = g.nx / 2, hz = g.nz / 2;
  const int64_t total = (int64_t)g.B * h * g.nx * g.nz;
  const int64_t stride = (int64_t)g.NX * g.NZ;
  double acc = 0.0;
  for (int64_t t = blockIdx.x * (int64_t)blockDim.x + threadIdx.x; t < total; t += (int64_t)gridDim.x * blockDim.x) {
    const int n = (int)(t % g.nz);
    int64_t r = t / g.nz;
    const int x = (int)(r % g.nx);
    r /= g.nx;
    const int i = (int)(r % h);
    const int b = (int)(r / h);
    const int64_t base = dt3_off(g, b, 0, x, n);
    float2 lo[8], hi[8];
#pragma unroll
    for (int k = 0; k < 8; ++k) afb_line(J.f[k], J.src[k] + base, stride, g.ny, i, lo[k], hi[k]);
    const bool low3 = n < hz && x < hx;   // y-low output of the all-low band continues to the next level
    if (!low3) dt3_group<SHRINK>(lo, tau2, acc);
    dt3_group<SHRINK>(hi, tau2, acc);
#pragma unroll
    for (int k = 0; k < 8; ++k) {
      if (SHRINK || low3) J.dst[k][base + (int64_t)i * stride] = lo[k];
      if (SHRINK) J.dst[k][base + (int64_t)(h + i) * stride] = hi[k];
    }
  }
  if (!SHRINK) {
#pragma unroll
    for (int o = 32; o > 0; o >>= 1) acc += __shfl_xor(acc, o);
    const int lane = threadIdx.x & 63, w = threadIdx.x >> 6;
    if (lane == 0) sh[w] = acc;
    __syncthreads();
    if (threadIdx.x == 0) {
      double s = 0.0;
      for (int k = 0; k < (int)(blockDim.x >> 6); ++k) s += sh[k];
      partial[blockIdx.x] = s;
    }
  }
}

// The first level's y analysis with a sliding register window: there the
// eight trees read four sources (trees 2q and 2q + 1 filter the same staging
// buffer with the two filters), and output i reads rows 2i .. 2i + NT - 1,
// so a thread walking RP outputs along y (one depth lane, one x) keeps NT
// rows of each source in registers and loads two new rows per output.  Taps
// in afb_line's order: the coefficients, and every value written, are those
// of afb3_y8_kernel bit for bit (the value pass's FP64 partial sums add the
// same terms in another order).
template <bool SHRINK, int NT>
__global__ void __launch_bounds__(256) afb3_y8_window(Dt3Geom g, DtJobs8 J, float tau2, double* partial) {
  constexpr int RP = 16;
  __shared__ double sh[16];
  const int len = g.ny, h = g.ny / 2, hx = g.nx / 2, hz = g.nz / 2;
  const int runs = (h + RP - 1) / RP;
  const int64_t total = (int64_t)g.B * runs * g.nx * g.nz;
  const int64_t stride = (int64_t)g.NX * g.NZ;
  double acc = 0.0;
  for (int64_t t = blockIdx.x * (int64_t)blockDim.x + threadIdx.x; t < total; t += (int64_t)gridDim.x * blockDim.x) {
    const int n = (int)(t % g.nz);
    int64_t r = t / g.nz;
    const int x = (int)(r % g.nx);
    r /= g.nx;
    const int run = (int)(r % runs);
    const int b = (int)(r / runs);
    const int64_t base = dt3_off(g, b, 0, x, n);
    const int i0 = run * RP;
    const bool low3 = n < hz && x < hx;   // y-low output of the all-low band continues to the next level
    // slot u % NT holds row (2 i0 + u) mod len of source q (trees 2q, 2q + 1)
    float2 win[4][NT];
#pragma unroll
    for (int u = 0; u < NT - 2; ++u) {
      const int row = (2 * i0 + u) % len;
#pragma unroll
      for (int q = 0; q < 4; ++q) win[q][u % NT] = J.src[2 * q][base + (int64_t)row * stride];
    }
#pragma unroll
    for (int si = 0; si < RP; ++si) {
      const int i = i0 + si;
      if (i < h) {
#pragma unroll
        for (int e = 0; e < 2; ++e) {
          const int u = 2 * si + NT - 2 + e;
          const int row = (2 * i0 + u) % len;
#pragma unroll
          for (int q = 0; q < 4; ++q) win[q][u % NT] = J.src[2 * q][base + (int64_t)row * stride];
        }
        float2 lo[8], hi[8];
#pragma unroll
        for (int k8 = 0; k8 < 8; ++k8) {
          const DtFilt& f = J.f[k8];
          lo[k8] = make_float2(0.f, 0.f);
          hi[k8] = make_float2(0.f, 0.f);
#pragma unroll
          for (int k = 0; k < NT; ++k) {
            const float2 v = win[k8 >> 1][(2 * si + k) % NT];
            fma2(lo[k8], f.h0[k], v);
            fma2(hi[k8], f.h1[k], v);
          }
        }
        if (!low3) dt3_group<SHRINK>(lo, tau2, acc);
        dt3_group<SHRINK>(hi, tau2, acc);
#pragma unroll
        for (int k8 = 0; k8 < 8; ++k8) {
          if (SHRINK || low3) J.dst[k8][base + (int64_t)i * stride] = lo[k8];
          if (SHRINK) J.dst[k8][base + (int64_t)(h + i) * stride] = hi[k8];
        }
      }
    }
  }
  if (!SHRINK) {
#pragma unroll
    for (int o = 32; o > 0; o >>= 1) acc += __shfl_xor(acc, o);
    const int lane = threadIdx.x & 63, w = threadIdx.x >> 6;
    if (lane == 0) sh[w] = acc;
    __syncthreads();
    if (threadIdx.x == 0) {
      double s = 0.0;
      for (int k = 0; k < (int)(blockDim.x >> 6); ++k) s += sh[k];
      partial[blockIdx.x] = s;
    }
  }
}

// x analysis with a sliding register window (one job per blockIdx.y, one
// source and one filter each): output i reads rows 2i .. 2i + NT - 1.
template <int NT>
__global__ void __launch_bounds__(256) afb3_x_window(Dt3Geom g, DtJobs8 J) {
  constexpr int RP = 16;
  const int j = blockIdx.y;
  const DtFilt& f = J.f[j];
  const int len = g.nx, h = g.nx / 2;
  const int runs = (h + RP - 1) / RP;
  const int64_t total = (int64_t)g.B * g.ny * runs * g.nz;
  const int64_t stride = g.NZ;
  for (int64_t t = blockIdx.x * (int64_t)blockDim.x + threadIdx.x; t < total; t += (int64_t)gridDim.x * blockDim.x) {
    const int n = (int)(t % g.nz);
    int64_t r = t / g.nz;
    const int run = (int)(r % runs);
    r /= runs;
    const int y = (int)(r % g.ny);
    const int b = (int)(r / g.ny);
    const int64_t base = dt3_off(g, b, y, 0, n);
    const int i0 = run * RP;
    float2 win[NT];
#pragma unroll
    for (int u = 0; u < NT - 2; ++u) win[u % NT] = J.src[j][base + (int64_t)((2 * i0 + u) % len) * stride];
#pragma unroll
    for (int si = 0; si < RP; ++si) {
      const int i = i0 + si;
      if (i < h) {
#pragma unroll
        for (int e = 0; e < 2; ++e) {
          const int u = 2 * si + NT - 2 + e;
          win[u % NT] = J.src[j][base + (int64_t)((2 * i0 + u) % len) * stride];
        }
        float2 lo = make_float2(0.f, 0.f), hi = make_float2(0.f, 0.f);
#pragma unroll
        for (int k = 0; k < NT; ++k) {
          const float2 v = win[(2 * si + k) % NT];
          fma2(lo, f.h0[k], v);
          fma2(hi, f.h1[k], v);
        }
        J.dst[j][base + (int64_t)i * stride] = lo;
        J.dst[j][base + (int64_t)(h + i) * stride] = hi;
      }
    }
  }
}

// Workspace of the volume transform: 8 trees, then staging buffers S (8) and
// U (8), one image each.
struct Dt3Work {
  float2* tree[8];
  float2* S[8];
  float2* U[8];
};

Dt3Work dt3_work(float2* work, int64_t n) {
  Dt3Work w;
  for (int t = 0; t < 8; ++t) {
    w.tree[t] = work + t * n;
    w.S[t] = work + (8 + t) * n;
    w.U[t] = work + (16 + t) * n;
  }
  return w;
}

// Analysis of the eight trees; mode 0 shrinks the details by tau2, mode 1
// writes the block partials of sum |W x| (value pass).
hipError_t dt3_analysis(const Dt3Geom& g0, int levels, const float2* v, const Dt3Work& w, int mode, float tau2,
                        double* partial, hipStream_t s) {
  const DtFilters& F = filters();
  Dt3Geom g = g0;
  for (int lev = 0; lev < levels; ++lev) {
    const DtFilt* fs = lev == 0 ? F.first : F.later;
    DtJobs8 jz{}, jx{}, jy{};
    int nz_jobs, nx_jobs;
    if (lev == 0) {
      // depth filters once per depth tree, x filters once per (depth, x) pair
      nz_jobs = 2;
      for (int p = 0; p < 2; ++p) {
        jz.src[p] = v;
        jz.dst[p] = w.S[p];
        jz.f[p] = fs[p];
      }
      nx_jobs = 4;
      for (int p = 0; p < 4; ++p) {
        jx.src[p] = w.S[p >> 1];
        jx.dst[p] = w.U[p];
        jx.f[p] = fs[p & 1];
      }
      for (int t = 0; t < 8; ++t) {
        jy.src[t] = w.U[t >> 1];
        jy.dst[t] = w.tree[t];
        jy.f[t] = fs[t & 1];
      }
    } else {
      nz_jobs = nx_jobs = 8;
      for (int t = 0; t < 8; ++t) {
        jz.src[t] = w.tree[t];
        jz.dst[t] = w.S[t];
        jz.f[t] = fs[t >> 2];
        jx.src[t] = w.S[t];
        jx.dst[t] = w.U[t];
        jx.f[t] = fs[(t >> 1) & 1];
        jy.src[t] = w.U[t];
        jy.dst[t] = w.tree[t];
        jy.f[t] = fs[t & 1];
      }
    }
    const int64_t nzw = (int64_t)g.B * g.ny * g.nx * (g.nz / 2), nxw = (int64_t)g.B * g.ny * (g.nx / 2) * g.nz;
    const int64_t nyw = (int64_t)g.B * (g.ny / 2) * g.nx * g.nz;
    hipLaunchKernelGGL(afb3_kernel<0>, dim3(dt_grid_y(nzw, nz_jobs), nz_jobs), dim3(256), 0, s, g, jz);
    // x: register-window kernel for the 8- and 12-tap filters
    const int ntx = jx.f[0].n;
    const int64_t tw = (int64_t)g.B * g.ny * ((g.nx / 2 + 15) / 16) * g.nz;
    bool xw = (ntx == 8 || ntx == 12) && tw >= DT_WINDOW_MIN_THREADS;
    for (int q = 0; q < nx_jobs; ++q) xw = xw && jx.f[q].n == ntx;
    if (xw) {
      if (ntx == 8)
        hipLaunchKernelGGL(afb3_x_window<8>, dim3(dt_grid_y(tw, nx_jobs), nx_jobs), dim3(256), 0, s, g, jx);
      else
        hipLaunchKernelGGL(afb3_x_window<12>, dim3(dt_grid_y(tw, nx_jobs), nx_jobs), dim3(256), 0, s, g, jx);
    } else {
      hipLaunchKernelGGL(afb3_kernel<1>, dim3(dt_grid_y(nxw, nx_jobs), nx_jobs), dim3(256), 0, s, g, jx);
    }
    // y: at the first level the trees read four sources with two 8-tap filters: register window
    const bool yw = lev == 0 && fs[0].n == 8 && fs[1].n == 8 &&
                    (int64_t)g.B * ((g.ny / 2 + 15) / 16) * g.nx * g.nz >= DT_WINDOW_MIN_THREADS;
    if (mode == 0) {
      if (yw)
        hipLaunchKernelGGL((afb3_y8_window<true, 8>), dim3(dt_grid(nyw)), dim3(256), 0, s, g, jy, tau2, nullptr);
      else
        hipLaunchKernelGGL((afb3_y8_kernel<true>), dim3(dt_grid(nyw)), dim3(256), 0, s, g, jy, tau2, nullptr);
    } else {
      if (yw)
        hipLaunchKernelGGL((afb3_y8_window<false, 8>), dim3(dt_grid(nyw)), dim3(256), 0, s, g, jy, 0.f, partial);
      else
        hipLaunchKernelGGL((afb3_y8_kernel<false>), dim3(dt_grid(nyw)), dim3(256), 0, s, g, jy, 0.f, partial);
      partial += dt_grid(nyw);
    }
    g.ny /= 2;
    g.nx /= 2;
    g.nz /= 2;
  }
  return hipGetLastError();
}

}  // namespace

int dtcwt_partials(const ProxGeom& pg, int levels) {
  int n = 0;
  if (pg.lateral_dims == 2) {
    int64_t ny = pg.Ny, nx = pg.Nx, nz = pg.Nz;
    for (int lev = 0; lev < levels; ++lev) {
      n += dt_grid((int64_t)pg.B * (ny / 2) * nx * nz);
      ny /= 2;
      nx /= 2;
      nz /= 2;
    }
    return n;
  }
  for (int lev = 0; lev < levels; ++lev) n += (int)dt_analysis_grid(dt_level(pg, lev), lev);
  return n;
}

size_t dtcwt_work_elems(const ProxGeom& pg) {
  const size_t n = (size_t)pg.B * pg.Ny * pg.Nx * pg.Nz;
  return (pg.lateral_dims == 2 ? 24 : 8) * n;
}

// Lateral synthesis pass of the volume: the register-window kernel for the 8-
// and 12-tap filters on large enough sub-arrays, else the per-tap one.
template <int AXIS, bool ACC>
void sfb3_lateral(const Dt3Geom& g, const DtJobs8& J, int jobs, hipStream_t s) {
  const int nt = J.f[0].n;
  bool same = true;
  for (int q = 0; q < jobs * (ACC ? 2 : 1); ++q) same = same && J.f[q].n == nt;
  const int len = AXIS == 1 ? g.nx : g.ny, others = AXIS == 1 ? g.ny : g.nx;
  const int64_t total = (int64_t)g.B * others * ((len / 2 + 15) / 16) * g.nz;
  if (same && (nt == 8 || nt == 12) && total >= DT_WINDOW_MIN_THREADS) {
    if (nt == 8)
      hipLaunchKernelGGL((sfb3_window<AXIS, ACC, 8>), dim3(dt_grid_y(total, jobs), jobs), dim3(256), 0, s, g, J);
    else
      hipLaunchKernelGGL((sfb3_window<AXIS, ACC, 12>), dim3(dt_grid_y(total, jobs), jobs), dim3(256), 0, s, g, J);
    return;
  }
  const int64_t nn = (int64_t)g.B * g.ny * g.nx * g.nz;
  hipLaunchKernelGGL((sfb3_kernel<AXIS, ACC>), dim3(dt_grid_y(nn, jobs), jobs), dim3(256), 0, s, g, J);
}

hipError_t launch_prox_dtcwt3(const ProxGeom& pg, int levels, const float2* v, float2* z, float tau, float2* work,
                              hipStream_t s) {
  const int64_t n = (int64_t)pg.B * pg.Ny * pg.Nx * pg.Nz;
  const Dt3Work w = dt3_work(work, n);
  const Dt3Geom g0{pg.B, pg.Ny, pg.Nx, pg.Nz, pg.Ny, pg.Nx, pg.Nz};
  // unscaled trees: soft threshold 2^(3/2) tau, synthesis sum scaled by 1/8
  hipError_t e = dt3_analysis(g0, levels, v, w, 0, 2.8284271247461900976f * tau, nullptr, s);
  if (e != hipSuccess) return e;
  const DtFilters& F = filters();
  for (int lev = levels - 1; lev >= 0; --lev) {
    Dt3Geom gl = g0;
    gl.ny = pg.Ny >> lev;
    gl.nx = pg.Nx >> lev;
    gl.nz = pg.Nz >> lev;
    const DtFilt* fs = lev == 0 ? F.first : F.later;
    const int64_t nn = (int64_t)gl.B * gl.ny * gl.nx * gl.nz;
    DtJobs8 jy{}, jx{}, jz{};
    jy.scale = jx.scale = jz.scale = 1.f;
    if (lev > 0) {
      for (int t = 0; t < 8; ++t) {
        jy.src[t] = w.tree[t];
        jy.dst[t] = w.S[t];
        jy.f[t] = fs[t & 1];
        jx.src[t] = w.S[t];
        jx.dst[t] = w.U[t];
        jx.f[t] = fs[(t >> 1) & 1];
        jz.src[t] = w.U[t];
        jz.dst[t] = w.tree[t];
        jz.f[t] = fs[t >> 2];
      }
      sfb3_lateral<2, false>(gl, jy, 8, s);
      sfb3_lateral<1, false>(gl, jx, 8, s);
      hipLaunchKernelGGL((sfb3_kernel<0, false>), dim3(dt_grid_y(nn, 8), 8), dim3(256), 0, s, gl, jz);
    } else {
      // y: trees (p, ty = a) + (p, ty = b) -> S[2q], p = 4 tz + 2 tx = 2q; x: S[4 tz] + S[4 tz + 2] -> U[tz];
      // depth: U[a] + U[b], times 1/8, -> z
      for (int t = 0; t < 8; ++t) {
        jy.src[t] = w.tree[t];
        jy.dst[t] = w.S[t];
        jy.f[t] = fs[t & 1];
      }
      for (int q = 0; q < 4; ++q) {
        jx.src[q] = w.S[2 * q];
        jx.dst[q] = w.U[q];
        jx.f[q] = fs[q & 1];
      }
      jz.src[0] = w.U[0];
      jz.src[1] = w.U[2];
      jz.dst[0] = z;
      jz.f[0] = fs[0];
      jz.f[1] = fs[1];
      jz.scale = 0.125f;
      sfb3_lateral<2, true>(gl, jy, 4, s);
      sfb3_lateral<1, true>(gl, jx, 2, s);
      hipLaunchKernelGGL((sfb3_kernel<0, true>), dim3(dt_grid_y(nn, 1), 1), dim3(256), 0, s, gl, jz);
    }
  }
  return hipGetLastError();
}

hipError_t launch_prox_dtcwt(const ProxGeom& pg, int levels, const float2* v, float2* z, float tau, float2* work,
                             hipStream_t s) {
  if (pg.lateral_dims == 2) return launch_prox_dtcwt3(pg, levels, v, z, tau, work, s);
  // unscaled trees: soft threshold 2 tau, synthesis sum scaled by 1/4
  hipError_t e = dt_analysis(pg, levels, v, work, 0, 2.f * tau, nullptr, s);
  if (e != hipSuccess) return e;
  return dt_synthesis(pg, levels, z, work, s);
}

hipError_t launch_dtcwt_value(const ProxGeom& pg, int levels, const float2* x, float2* work, double* partial,
                              hipStream_t s) {
  if (pg.lateral_dims == 2) {
    const int64_t n = (int64_t)pg.B * pg.Ny * pg.Nx * pg.Nz;
    const Dt3Geom g0{pg.B, pg.Ny, pg.Nx, pg.Nz, pg.Ny, pg.Nx, pg.Nz};
    return dt3_analysis(g0, levels, x, dt3_work(work, n), 1, 0.f, partial, s);
  }
  return dt_analysis(pg, levels, x, work, 1, 0.f, partial, s);
}

// Host copies of the designed filters (for the library's own checks).
void dtcwt_filter_taps(int which, float* h0, int* n) {
  const DtFilters& F = filters();
  const DtFilt& f = which == 0 ? F.first[0] : which == 1 ? F.first[1] : which == 2 ? F.later[0] : F.later[1];
  *n = f.n;
  for (int k = 0; k < f.n; ++k) h0[k] = f.h0[k];
}
