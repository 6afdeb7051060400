// Column pairs of the ISAM resampling (Sec. 2.1, eq. (5)-(6)) on a grid
// oversampled exactly twice, K = 2 N (N = n_depth): the forward NUFFT, its
// adjoint, and both with the residual spectrum between them, for the columns
// q and -q of a half-spectrum slot (the pair kernels of oct_nufft.hip serve
// every other oversampling).  Against those kernels:
//
// * Grid transforms.  The even cells of the K-point transform of a zero-padded
//   column x are the N-point DFT of x, the odd cells the N-point DFT of
//   x e^{-i pi n'/N} (n' = n - n_c): four N-point rows per pair instead of two
//   K-point ones, with no zeros to transform, for every N that col_plan can
//   split.  Radices up to 16 leave two or three stages (two LDS exchanges at
//   2048, where radix 8 on 4096 points took three).  The first forward stage
//   reads the column from memory once for both rows, the last inverse stage
//   joins them into it.
// * Samples by grid cell.  Consecutive samples are at least one cell apart
//   (t' >= K dz dk / pi), and the host takes these kernels where a cell is the
//   base cell of at most one sample.  A thread owns SPT consecutive base cells, finds the
//   sample of each by inverting t(m), and its windows overlap: SPT + J - 1
//   cells are read, and added to, for SPT samples (J SPT of each before), the
//   weights serve both directions, and the adjoint needs no pass per tap: a
//   thread adds its samples up in registers, passes what falls beyond its own
//   cells to the next lanes, and writes every cell once.
//
// Bound by vector arithmetic on large launches of the compiled lengths: 17.7 k
// vector instructions per pair of 2048-point columns, 0.78 of the issue rate
// (23.2 k at 0.69 in the pair kernel).  At run-time lengths the stage switch, LDS
// and barriers leave 0.32 of it (1400 x 1120: 561 pairs on 512 resident
// workgroups, a second round of 49), and a few pairs are one pair's chain of
// barriers.  Both directions in one launch, pair kernel -> here: 2048 x 256 x 256
// 1.90 -> 1.30 ms, 32 x 1024 x 512 311 -> 167 us, 1400 x 1120 79 -> 39 us, 512 x
// 64 15.2 -> 9.2 us; the adjoint of 1024 x 112 x 112 145 -> 69 us, forward and
// adjoint of 2048 x 1000 17.2 and 21.5 -> 16.5 and 15.3 us.
#include "oct_fft.h"

#include <algorithm>
#include <cmath>
#include <vector>

namespace {

constexpr int KBH = (OCT_KB_DEG + 1) / 2;
constexpr int COL_PADK = 8;    // wrapped cells after each row
constexpr double COL_EPS = 0x1p-13;   // 1.2e-4; 1 - COL_EPS is exact

// Base cell of t: floor(t + COL_EPS), which no two samples of a column share
// where col_cells_distinct says so.  The q = 0 coordinates t_0 + h m (h >= 1
// cells apart) are integers for the usual optics, and a boundary at the integers
// would fall between cells by rounding; COL_EPS below them it does not.  The
// window's value COL_EPS beyond its edge is below 4e-8 of its peak (J = 6).

__device__ __forceinline__ double col_sqrt(double arg) {   // arg > 0; relative error ~2e-14
  const double r0 = (double)__builtin_amdgcn_rsqf(fmaxf((float)arg, 1e-30f));
  const double h = arg * r0;
  return fma(0.5 * h, fma(-h, r0, 1.0), h);
}

__device__ __forceinline__ int padk(int i) { return i + (i >> 4); }   // spreads strided LDS accesses over the banks

// Runtime lengths: only a first stage whose radix is a multiple of 4 leaves the
// padded layout (other strides meet at most two lanes in a bank); everything
// else is natural, one addition per access instead of four operations.
template <int R, int CN>
__device__ __forceinline__ int col_first_w(int j, int r);

// padk(base + r NS) for a stage's writes, with constant offsets where base's
// low bits are known
template <int R, int NS>
__device__ __forceinline__ int pad_w(int base, int r) {
  if constexpr (NS > 0 && NS % 16 == 0) return padk(base) + r * (NS + NS / 16);
  else if constexpr (NS == 8 && R % 2 == 0) return padk(base) + 8 * r + (r >> 1);   // base mod 16 < 8
  else if constexpr (NS == 1 && (R == 8 || R == 16)) return padk(base) + r;         // base = R j
  else return padk(base + r * NS);
}
// padk(j + r nb)
template <int NB>
__device__ __forceinline__ int pad_r(int j, int r, int nb) {
  if constexpr (NB > 0 && NB % 16 == 0) return padk(j) + r * (NB + NB / 16);
  else return padk(j + r * nb);
}

template <int R, int CN>
__device__ __forceinline__ int col_first_w(int j, int r) {   // where a first stage writes output r of butterfly j
  if constexpr (CN != 0 || R % 4 == 0) return pad_w<R, 1>(j * R, r);
  else return j * R + r;
}

template <int R, bool INV>
__device__ __forceinline__ void col_twiddle(float2* v, const float2* __restrict__ tw, int k) {
  constexpr int NQ = fft_tw_pad(R) / 2;
  const float4* __restrict__ tp = reinterpret_cast<const float4*>(tw) + k * NQ;
  float4 q[NQ];
#pragma unroll
  for (int i = 0; i < NQ; ++i) q[i] = tp[i];
#pragma unroll
  for (int r = 1; r < R; ++r) {
    const float4 f = q[(r - 1) >> 1];
    float2 w = ((r - 1) & 1) ? make_float2(f.z, f.w) : make_float2(f.x, f.y);
    if (INV) w.y = -w.y;
    v[r] = cmul(v[r], w);
  }
}

// LDS: cell (parity, i) of column c at g[(parity rs + i) 2 + c]
struct ColLds {
  float2* g;
  int rs;
  __device__ __forceinline__ float2* row(int par, int c) const { return g + 2 * par * rs + c; }
};

// First forward stage: butterfly j of column c, rows even and odd, from memory.
template <int R, int CN>
__device__ __forceinline__ void col_fwd_first(const ColArgs& a, const ColLds& l, const float2* s0, const float2* s1,
                                              int tid, int nthr) {
  const int N = CN ? CN : a.Nz, nc = CN ? CN / 2 : a.nc;
  const int nb = N / R;
  for (int item = tid; item < 2 * nb; item += nthr) {
    const int c = item & 1, j = item >> 1;
    const float2* __restrict__ src = c ? s1 : s0;
    float2 x[R], v[R];
    float d[R];
    auto depth = [&](int r) __attribute__((always_inline)) {
      const int n = j + r * nb + nc;
      return n >= N ? n - N : n;
    };
#pragma unroll
    for (int r = 0; r < R; ++r) {
      x[r] = src[depth(r)];
      d[r] = a.deap[depth(r)];
    }
#pragma unroll
    for (int r = 0; r < R; ++r) v[r] = cscale(x[r], d[r]);
    Dft<R, false>::run(v);
    float2* dst = l.row(0, c);
#pragma unroll
    for (int r = 0; r < R; ++r) dst[2 * col_first_w<R, CN>(j, r)] = v[r];
#pragma unroll
    for (int r = 0; r < R; ++r) v[r] = cmul(x[r], a.deap_odd[depth(r)]);
    Dft<R, false>::run(v);
    dst = l.row(1, c);
#pragma unroll
    for (int r = 0; r < R; ++r) dst[2 * col_first_w<R, CN>(j, r)] = v[r];
  }
  __syncthreads();
}

// A stage in place over the four rows, up to MB butterflies per thread.
// FIRST: the inverse's first stage (natural input).  LAST: the forward's last
// (natural output, and the wrapped cells after each row).  pin (runtime
// lengths): the input is padded.
template <int R, int MB, int CN, int CNS, bool INV, bool FIRST, bool LAST>
__device__ __forceinline__ void col_stage(const ColLds& l, int n, int ns, const FastDiv& dns,
                                          const float2* __restrict__ tw, bool pin, int tid, int nthr) {
  const int N = CN ? CN : n, Ns = CNS ? CNS : ns;
  const int nb = N / R;
  // opaque: the addresses of every radix in the stage loop's switch would
  // otherwise be formed ahead of the loop (70-150 spilled registers)
  if (CN == 0) asm volatile("" : "+v"(tid));
  float2 v[MB][R];
  int base[MB], par[MB];
#pragma unroll
  for (int b = 0; b < MB; ++b) {
    const int c = (tid + b * nthr) & 1, q = (tid + b * nthr) >> 1;
    if (q < 2 * nb) {
      par[b] = q >= nb ? 1 : 0;
      const int j = q - par[b] * nb;
      const int k = FIRST ? 0 : CNS ? j % CNS : j - (int)fdiv((uint32_t)j, dns) * Ns;
      const float2* src = l.row(par[b], c);
      if (FIRST || (CN == 0 && !pin)) {
        const float2* s = src + 2 * j;
#pragma unroll
        for (int r = 0; r < R; ++r) v[b][r] = s[2 * r * nb];
      } else {
#pragma unroll
        for (int r = 0; r < R; ++r) v[b][r] = src[2 * pad_r<CN / R>(j, r, nb)];
      }
      if (!FIRST) col_twiddle<R, INV>(v[b], tw, k);
      Dft<R, INV>::run(v[b]);
      base[b] = FIRST ? j : (j - k) * R + k;
    }
  }
  __syncthreads();
#pragma unroll
  for (int b = 0; b < MB; ++b) {
    const int c = (tid + b * nthr) & 1, q = (tid + b * nthr) >> 1;
    if (q < 2 * nb) {
      float2* dst = l.row(par[b], c);
      if (FIRST) {
#pragma unroll
        for (int r = 0; r < R; ++r) dst[2 * col_first_w<R, CN>(base[b], r)] = v[b][r];
      } else if (LAST || CN == 0) {
        float2* d = dst + 2 * base[b];
#pragma unroll
        for (int r = 0; r < R; ++r) d[2 * r * Ns] = v[b][r];
        if (LAST && base[b] < COL_PADK) dst[2 * (N + base[b])] = v[b][0];   // base = k < Ns, Ns >= COL_PADK
      } else {
#pragma unroll
        for (int r = 0; r < R; ++r) dst[2 * pad_w<R, CNS>(base[b], r)] = v[b][r];
      }
    }
  }
  __syncthreads();
}

// Last inverse stage: both rows of column c, joined and deapodised into memory.
template <int R, int CN>
__device__ __forceinline__ void col_inv_last(const ColArgs& a, const ColLds& l, const float2* __restrict__ tw,
                                             bool pin, float2* d0, float2* d1, int tid, int nthr) {
  const int N = CN ? CN : a.Nz, nc = CN ? CN / 2 : a.nc;
  const int nb = N / R;   // = Ns
  for (int item = tid; item < 2 * nb; item += nthr) {
    const int c = item & 1, j = item >> 1;
    float2* __restrict__ dst = c ? d1 : d0;
    if (!dst) continue;
    float2 v[R], w[R];
    const float2 *ra = l.row(0, c), *rb = l.row(1, c);
    if (CN == 0 && !pin) {
      const float2 *sa = ra + 2 * j, *sb = rb + 2 * j;
#pragma unroll
      for (int r = 0; r < R; ++r) {
        v[r] = sa[2 * r * nb];
        w[r] = sb[2 * r * nb];
      }
    } else {
#pragma unroll
      for (int r = 0; r < R; ++r) {
        const int o = 2 * pad_r<CN / R>(j, r, nb);
        v[r] = ra[o];
        w[r] = rb[o];
      }
    }
    col_twiddle<R, true>(v, tw, j);
    Dft<R, true>::run(v);
    col_twiddle<R, true>(w, tw, j);
    Dft<R, true>::run(w);
#pragma unroll
    for (int r = 0; r < R; ++r) {
      int n = j + r * nb + nc;
      if (n >= N) n -= N;
      const float d = a.deap[n];
      const float2 e = a.deap_odd[n];
      const float2 o = cmul(w[r], cconj(e));
      dst[n] = make_float2(fmaf(d, v[r].x, o.x), fmaf(d, v[r].y, o.y));
    }
  }
}

// ---- the transforms, compile-time lengths (plans of col_plan: 512 = 8 8 8,
// 1024 = 8 8 16, 2048 = 8 16 16) or any planned length (CN = 0)
#define COL_RADIX_SWITCH(radix, CALL) \
  switch (radix) {                    \
    case 4: CALL(4); break;           \
    case 5: CALL(5); break;           \
    case 6: CALL(6); break;           \
    case 7: CALL(7); break;           \
    case 8: CALL(8); break;           \
    case 9: CALL(9); break;           \
    case 10: CALL(10); break;         \
    case 12: CALL(12); break;         \
    case 14: CALL(14); break;         \
    case 15: CALL(15); break;         \
    default: CALL(16); break;         \
  }

// the stages that touch memory hold two rows per thread: radices up to 12
#define COL_EDGE_SWITCH(radix, CALL) \
  switch (radix) {                   \
    case 4: CALL(4); break;          \
    case 5: CALL(5); break;          \
    case 6: CALL(6); break;          \
    case 7: CALL(7); break;          \
    case 8: CALL(8); break;          \
    case 9: CALL(9); break;          \
    case 10: CALL(10); break;        \
    default: CALL(12); break;        \
  }

template <int CN, int MB>
__device__ __forceinline__ void col_forward(const ColArgs& a, const ColLds& l, const float2* s0, const float2* s1,
                                            int tid, int nthr) {
  const FastDiv none{};
  if constexpr (CN == 512 || CN == 1024 || CN == 2048) {
    constexpr int R1 = CN == 2048 ? 16 : 8, R2 = CN == 512 ? 8 : 16;
    col_fwd_first<8, CN>(a, l, s0, s1, tid, nthr);
    col_stage<R1, MB, CN, 8, false, false, false>(l, CN, 8, none, a.tw + a.f.tw_off[1], true, tid, nthr);
    col_stage<R2, MB, CN, 8 * R1, false, false, true>(l, CN, 8 * R1, none, a.tw + a.f.tw_off[2], true, tid, nthr);
  } else {
#define COL_FIRST(R) col_fwd_first<R, 0>(a, l, s0, s1, tid, nthr)
    COL_EDGE_SWITCH(a.f.radix[0], COL_FIRST)
#undef COL_FIRST
    const int last = a.f.ns - 1;
    const bool pad = a.f.radix[0] % 4 == 0;
    for (int s = 1; s < last; ++s) {
#define COL_MID(R) \
  col_stage<R, MB, 0, 0, false, false, false>(l, a.Nz, a.f.sub[s], a.f.div_sub[s], a.tw + a.f.tw_off[s], \
                                              s == 1 && pad, tid, nthr)
      COL_RADIX_SWITCH(a.f.radix[s], COL_MID)
#undef COL_MID
    }
#define COL_LAST(R) \
  col_stage<R, MB, 0, 0, false, false, true>(l, a.Nz, a.f.sub[last], a.f.div_sub[last], a.tw + a.f.tw_off[last], \
                                             last == 1 && pad, tid, nthr)
    COL_RADIX_SWITCH(a.f.radix[last], COL_LAST)
#undef COL_LAST
  }
}

template <int CN, int MB>
__device__ __forceinline__ void col_inverse(const ColArgs& a, const ColLds& l, float2* d0, float2* d1, int tid,
                                            int nthr) {
  const FastDiv none{};
  if constexpr (CN == 512 || CN == 1024 || CN == 2048) {
    constexpr int R0 = CN == 512 ? 8 : 16, R1 = CN == 2048 ? 16 : 8;
    col_stage<R0, MB, CN, 1, true, true, false>(l, CN, 1, none, a.tw, false, tid, nthr);
    col_stage<R1, MB, CN, R0, true, false, false>(l, CN, R0, none, a.tw + a.i.tw_off[1], true, tid, nthr);
    col_inv_last<8, CN>(a, l, a.tw + a.i.tw_off[2], true, d0, d1, tid, nthr);
  } else {
    const FastDiv one = a.i.div_sub[0];
#define COL_FIRST(R) col_stage<R, MB, 0, 0, true, true, false>(l, a.Nz, 1, one, a.tw, false, tid, nthr)
    COL_RADIX_SWITCH(a.i.radix[0], COL_FIRST)
#undef COL_FIRST
    const int last = a.i.ns - 1;
    const bool pad = a.i.radix[0] % 4 == 0;
    for (int s = 1; s < last; ++s) {
#define COL_MID(R) \
  col_stage<R, MB, 0, 0, true, false, false>(l, a.Nz, a.i.sub[s], a.i.div_sub[s], a.tw + a.i.tw_off[s], \
                                             s == 1 && pad, tid, nthr)
      COL_RADIX_SWITCH(a.i.radix[s], COL_MID)
#undef COL_MID
    }
#define COL_LAST(R) col_inv_last<R, 0>(a, l, a.tw + a.i.tw_off[last], last == 1 && pad, d0, d1, tid, nthr)
    COL_EDGE_SWITCH(a.i.radix[last], COL_LAST)
#undef COL_LAST
  }
}

__device__ __forceinline__ float from_prev_lane(float v) {   // 0 in lane 0
  return __int_as_float(__builtin_amdgcn_mov_dpp(__float_as_int(v), 0x138, 0xf, 0xf, true));
}

__device__ __forceinline__ void fma4(float4& s, float w, float4 v) {
  s.x = fmaf(w, v.x, s.x);
  s.y = fmaf(w, v.y, s.y);
  s.z = fmaf(w, v.z, s.z);
  s.w = fmaf(w, v.w, s.w);
}
__device__ __forceinline__ void add4(float4& s, float4 v) {
  s.x += v.x;
  s.y += v.y;
  s.z += v.z;
  s.w += v.w;
}

// p[i] by a 32-bit byte offset from a uniform base (no 64-bit address arithmetic per lane)
__device__ __forceinline__ float2 at32(const float2* p, int i) {
  return *reinterpret_cast<const float2*>(reinterpret_cast<const char*>(p) + (uint32_t)i * 8u);
}

enum { COL_FWD = 0, COL_ADJ = 1, COL_NORMAL = 2 };

// MODE COL_FWD: X (read) -> W_h(q) = (W(q) + conj W(-q)) / 2 in W.
// COL_ADJ: the spectra in W (read) -> both columns of X.
// COL_NORMAL: X -> R^ = W_h / N_lat - yh -> X (a pair reads its columns before
// it writes them), the pair's share of ||r||^2 by Parseval into r.partial.
// Up to MB butterflies per thread in the stages that run in place.
template <int J, int MODE, int CN, int SPT, int MB>
__global__ void __launch_bounds__(CN && SPT != 2 ? 512 : 1024, 4) column_pair_kernel(ColArgs a, const float2* X, float2* W,
                                                                       PairRes pr, float2* Xo) {
  extern __shared__ float4 smem4[];
  __shared__ float4 edge[16][J - 1];
  __shared__ double sh[16];
  const int tid = threadIdx.x, nthr = blockDim.x;
  const int lane = tid & 63, wave = __builtin_amdgcn_readfirstlane(tid >> 6);
  const int N = CN ? CN : a.Nz, K = 2 * N, Mk = a.Mk;
  const int b = blockIdx.x / a.n_pairs;
  const int4 pq = a.pairs[blockIdx.x - b * a.n_pairs];
  const ColSpan sp = a.spans[blockIdx.x - b * a.n_pairs];
  const int64_t item = (int64_t)b * a.item_cols;
  const int64_t col0 = (item + sp.x0) * N, col1 = (item + sp.x1) * N;
  const int64_t slot = ((int64_t)b * a.n_half + pq.z) * Mk;
  const ColLds l{reinterpret_cast<float2*>(smem4), a.rs};

  if constexpr (MODE != COL_ADJ) col_forward<CN, MB>(a, l, X + col0, X + col1, tid, nthr);

  // the base cells u0 .. u0 + SPT - 1 of this thread and their samples
  const double q2 = sp.q2;
  const float bq = sp.beam;
  const double ct = a.ct, k2min = 2.0 * a.k_min, dk2 = 2.0 * a.dk;
  auto coord = [&](double m) __attribute__((always_inline)) {   // t(m); not positive for evanescent samples
    const double k = fma(m, dk2, k2min);
    return ct * col_sqrt(fma(k, k, -q2));
  };
  const int o0 = SPT * tid;   // first own cell, counted from the window start of sp.umin
  const int u0 = sp.umin + o0;
  int cw = sp.cell0 + o0;     // window start of u0, in [0, K) wherever it is used (o0 < K)
  if (cw >= K) cw -= K;
  const int par = cw & 1, kap = cw >> 1;

  float4 own[SPT + J - 1];    // the adjoint's sums over the window
#pragma unroll
  for (int i = 0; i < SPT + J - 1; ++i) own[i] = make_float4(0.f, 0.f, 0.f, 0.f);
  double acc = 0.0;
  if (u0 <= sp.umax) {
    int m[SPT];
    float x[SPT];
    bool in[SPT];
    const double ict = a.inv_ct, hik = 0.5 * a.inv_dk, k0 = -a.k_min * a.inv_dk;
    const double ub = (double)u0, bt0 = (ub + (0.5 - COL_EPS)) * ict, mlast = (double)(Mk - 1);
    double md[SPT], d[SPT];
    float2 ph[SPT], rv[SPT];
    bool again = false;
    auto find = [&](int i) __attribute__((always_inline)) {   // is sample md[i] in cell u0 + i?
      const double t = coord(md[i]);
      d[i] = t - (ub + (double)i);   // exact
      in[i] = d[i] >= -COL_EPS && d[i] < 1.0 - COL_EPS && t > 0.0;
    };
#pragma unroll
    for (int i = 0; i < SPT; ++i) {
      // the only sample whose base cell can be u: the one nearest the cell's middle
      const double bt = fma((double)i, ict, bt0);
      md[i] = fmin(fmax(rint(fma(col_sqrt(fma(bt, bt, q2)), hik, k0)), 0.0), mlast);
      find(i);
      again |= !in[i] && fabsf((float)d[i] + (float)(COL_EPS - 0.5)) < 0.500002f;
    }
    if (again) {   // a rounding error past the cell's end: the sample at its other end is the one
#pragma unroll
      for (int i = 0; i < SPT; ++i) {
        const float off = (float)d[i] + (float)(COL_EPS - 0.5);
        if (!in[i] && fabsf(off) < 0.500002f) {
          md[i] = fmin(fmax(md[i] + (off < 0.f ? 1.0 : -1.0), 0.0), mlast);
          find(i);
        }
      }
    }
    const float2* __restrict__ rin = MODE == COL_ADJ ? W + slot : pr.yh ? pr.yh + slot : a.phase;
    const bool has_r = MODE == COL_ADJ || pr.yh;
#pragma unroll
    for (int i = 0; i < SPT; ++i) {
      m[i] = (int)md[i];
      x[i] = (float)fma(2.0, d[i], -1.0);
      ph[i] = at32(a.phase, m[i]);
      if constexpr (MODE != COL_FWD) {
        const float2 r = at32(rin, m[i]);
        rv[i] = make_float2(has_r ? r.x : 0.f, has_r ? r.y : 0.f);
      }
    }
    float w[SPT][J];
#pragma unroll
    for (int i = 0; i < SPT; ++i) {
      const float xs = in[i] ? x[i] : 0.f, x2 = xs * xs;   // an empty cell's weights only have to be finite
#pragma unroll
      for (int jj = 0; jj < J / 2; ++jj) {
        const float* __restrict__ c = a.kbc + jj * 2 * KBH;
        float e = c[KBH - 1], o = c[2 * KBH - 1];
#pragma unroll
        for (int d = KBH - 2; d >= 0; --d) {
          e = fmaf(e, x2, c[d]);
          o = fmaf(o, x2, c[KBH + d]);
        }
        w[i][jj] = fmaf(xs, o, e);
        w[i][J - 1 - jj] = fmaf(-xs, o, e);
      }
    }
    float4 v[SPT];
#pragma unroll
    for (int i = 0; i < SPT; ++i) v[i] = make_float4(0.f, 0.f, 0.f, 0.f);
    if constexpr (MODE != COL_ADJ) {
      // window cell i: even i in the row of cw's parity, odd i in the other
      const float4* ge = reinterpret_cast<const float4*>(l.g) + par * a.rs + kap;
      const float4* go = reinterpret_cast<const float4*>(l.g) + (par ? kap + 1 : a.rs + kap);
#pragma unroll
      for (int i = 0; i < SPT + J - 1; ++i) {
        const float4 g = (i & 1) ? go[i >> 1] : ge[i >> 1];
#pragma unroll
        for (int s = 0; s < SPT; ++s)
          if (i >= s && i - s < J) fma4(v[s], w[s][i - s], g);
      }
    }
    // the filter H(m, q) of the cells' samples (0 in empty cells)
    if (a.df != 0.0) {   // defocus phase, reduced modulo 2 pi in FP64
#pragma unroll
      for (int i = 0; i < SPT; ++i) {
        constexpr double two_pi = 6.283185307179586, inv_two_pi = 0.15915494309189535;
        // t of the cell's sample; what an empty cell looked at may be evanescent and give no finite phase
        const double phase = (in[i] ? coord((double)m[i]) : 0.0) * ict * a.df;
        const float f = (float)fma(-rint(phase * inv_two_pi), two_pi, phase);
        float sn, cs;
        sincosf(f, &sn, &cs);
        ph[i] = cmul(ph[i], make_float2(cs, sn));
      }
    }
#pragma unroll
    for (int i = 0; i < SPT; ++i) {
      const float g = in[i] ? bq : 0.f;
      ph[i] = make_float2(ph[i].x * g, ph[i].y * g);
      if constexpr (MODE != COL_ADJ) {
        const float2 w0 = cmul(ph[i], make_float2(v[i].x, v[i].y)), w1 = cmul(ph[i], make_float2(v[i].z, v[i].w));
        const float2 res = make_float2(0.5f * (w0.x + w1.x), 0.5f * (w0.y - w1.y));   // (W(q) + conj W(-q)) / 2
        if constexpr (MODE == COL_NORMAL)
          rv[i] = make_float2(fmaf(res.x, pr.inv_nlat, -rv[i].x), fmaf(res.y, pr.inv_nlat, -rv[i].y));
        else rv[i] = res;
      }
    }
    if constexpr (MODE == COL_FWD) {
      float2* __restrict__ out = W + slot;
#pragma unroll
      for (int i = 0; i < SPT; ++i)
        if (in[i]) out[m[i]] = rv[i];
      if (pq.w >= 0) {
        float2* __restrict__ outp = W + ((int64_t)b * a.n_half + pq.w) * Mk;
#pragma unroll
        for (int i = 0; i < SPT; ++i)
          if (in[i]) outp[m[i]] = cconj(rv[i]);
      }
    } else {
      if (MODE == COL_NORMAL && pr.partial) {
#pragma unroll
        for (int i = 0; i < SPT; ++i) {
          const double rx = in[i] ? rv[i].x : 0.f, ry = in[i] ? rv[i].y : 0.f;
          acc = fma(rx, rx, fma(ry, ry, acc));
        }
      }
#pragma unroll
      for (int i = 0; i < SPT; ++i) {
        const float2 hc = cconj(ph[i]);
        const float2 p0 = cmul(hc, rv[i]), p1 = cmul(hc, cconj(rv[i]));
        const float4 p = make_float4(p0.x, p0.y, p1.x, p1.y);
#pragma unroll
        for (int j = 0; j < J; ++j) fma4(own[i + j], w[i][j], p);
      }
    }
  }
  // evanescent samples (a prefix of the band, or all of it): W_h = 0, R^ = -yh with no column behind it
  if (MODE != COL_ADJ && sp.evan) {
    float2* __restrict__ out = W + slot;
    float2* __restrict__ outp = (MODE == COL_FWD && pq.w >= 0) ? W + ((int64_t)b * a.n_half + pq.w) * Mk : nullptr;
    for (int m = tid; m < Mk; m += nthr) {
      if (coord((double)m) > 0.0) continue;
      if constexpr (MODE == COL_FWD) {
        out[m] = make_float2(0.f, 0.f);
        if (outp) outp[m] = make_float2(0.f, 0.f);
      } else if (pr.partial && pr.yh) {
        const float2 y = pr.yh[slot + m];
        acc = fma((double)y.x, (double)y.x, fma((double)y.y, (double)y.y, acc));
      }
    }
  }
  if constexpr (MODE == COL_FWD) return;

  // what lies past the thread's own cells goes to the next lanes, past the
  // wave's to the next wave through `edge`
  float4 e[J - 1];
#pragma unroll
  for (int q = 0; q < J - 1; ++q) e[q] = make_float4(0.f, 0.f, 0.f, 0.f);
  if (sp.umin + SPT * 64 * wave <= sp.umax) {   // waves without samples have nothing to pass
    float4 cy[J - 1];
#pragma unroll
    for (int q = 0; q < J - 1; ++q) e[q] = cy[q] = own[SPT + q];
#pragma unroll
    for (int s = 0; s * SPT < J - 1; ++s) {   // s: lanes already passed
#pragma unroll
      for (int q = 0; q < J - 1 - s * SPT; ++q) {
        cy[q].x = from_prev_lane(cy[q].x);
        cy[q].y = from_prev_lane(cy[q].y);
        cy[q].z = from_prev_lane(cy[q].z);
        cy[q].w = from_prev_lane(cy[q].w);
      }
#pragma unroll
      for (int q = 0; q < J - 1 - s * SPT; ++q) {
        if (q < SPT) {
          add4(own[q], cy[q]);
        } else {
          cy[q - SPT] = cy[q];
          add4(e[q - SPT], cy[q]);   // lane 63: also on its way past the wave's end
        }
      }
    }
  }
  if (lane == 63) {
#pragma unroll
    for (int q = 0; q < J - 1; ++q) edge[wave][q] = e[q];
  }
  if (MODE == COL_NORMAL && pr.partial) {   // uniform
#pragma unroll
    for (int o = 32; o > 0; o >>= 1) acc += __shfl_xor(acc, o);
    if (lane == 0) sh[wave] = acc;
  }
  __syncthreads();   // the forward rows are read: the adjoint's take their place
  if (MODE == COL_NORMAL && pr.partial && tid == 0) {
    double t = 0.0;
    for (int w = 0; w < (nthr + 63) >> 6; ++w) t += sh[w];
    pr.partial[blockIdx.x] = t * pr.nlat * (pq.x != pq.y ? 2.0 : 1.0);
  }
  float4* rows = reinterpret_cast<float4*>(l.g);
  if (o0 < K) {
#pragma unroll
    for (int i = 0; i < SPT; ++i) {
      if (wave > 0 && lane * SPT + i < J - 1) add4(own[i], edge[wave - 1][lane * SPT + i]);
      if (o0 + i < K) {
        // cell cw + i, wrapped
        int r = ((par + i) & 1), kk = kap + ((par + i) >> 1);
        if (kk >= N) kk -= N;
        rows[r * a.rs + kk] = own[i];
      }
    }
  }
  for (int o = SPT * nthr + tid; o < K; o += nthr) {   // the cells no thread owns
    int c = sp.cell0 + o;
    if (c >= K) c -= K;
    rows[(c & 1) * a.rs + (c >> 1)] = make_float4(0.f, 0.f, 0.f, 0.f);
  }
  __syncthreads();
  col_inverse<CN, MB>(a, l, Xo + col0, pq.y != pq.x ? Xo + col1 : nullptr, tid, nthr);
}

// ns radices in increasing order: the first stage holds two rows per thread
// (radix <= 12), the others run in place with at most a butterfly for each of
// 1024 threads (no plan: 1750, 1875, 2000, a few more, most above 2048); the
// largest first radix wins (fewest butterflies)
bool plan_radices(int N, int ns, int* best) {
  constexpr int set[] = {4, 5, 6, 7, 8, 9, 10, 12, 14, 15, 16};
  bool found = false;
  int cur[4];
  auto rec = [&](auto&& self, int n, int s, int lo) -> void {
    if (s == ns) {
      if (n != 1) return;
      if (cur[0] > 12 || 4 * (N / cur[1]) > 1024 || N / cur[ns - 1] < COL_PADK) return;
      if (!found || std::lexicographical_compare(best, best + ns, cur, cur + ns)) std::copy(cur, cur + ns, best);
      found = true;
      return;
    }
    for (int r : set)
      if (r >= lo && n % r == 0) {
        cur[s] = r;
        self(self, n / r, s + 1, r);
      }
  };
  rec(rec, N, 0, 0);
  return found;
}

void fill_plan(int N, int ns, const int* radix, ColPlan* p, std::vector<float2>* tw) {
  p->ns = ns;
  int sub = 1;
  for (int s = 0; s < ns; ++s) {
    const int R = radix[s], P = fft_tw_pad(R);
    p->radix[s] = R;
    p->sub[s] = sub;
    p->div_sub[s] = make_fastdiv((uint32_t)sub);
    p->tw_off[s] = (int)tw->size();
    if (sub > 1)
      for (int k = 0; k < sub; ++k)
        for (int r = 1; r <= P; ++r) {
          const double ang = -2.0 * 3.14159265358979323846 * (double)(r * k) / (double)(sub * R);
          tw->push_back(r < R ? make_float2((float)std::cos(ang), (float)std::sin(ang)) : make_float2(0.f, 0.f));
        }
    sub *= R;
  }
}

template <int J, int MODE, int CN, int SPT, int MB>
hipError_t col_launch_t(const ColArgs& a, const float2* X, float2* W, const PairRes& r, float2* Xo, int nthr,
                        hipStream_t s) {
  const size_t lds = col_lds_bytes(a.Nz);
  if (lds > 48 * 1024) {
    // once per instantiation (thread-safe initialisation of a local static)
    static const hipError_t set =
        hipFuncSetAttribute(reinterpret_cast<const void*>(&column_pair_kernel<J, MODE, CN, SPT, MB>),
                            hipFuncAttributeMaxDynamicSharedMemorySize, 160 * 1024 - 4096);
    if (set != hipSuccess) return set;
  }
  hipLaunchKernelGGL((column_pair_kernel<J, MODE, CN, SPT, MB>), dim3(a.n_pairs * a.batch), dim3(nthr),
                     lds, s, a, X, W, r, Xo);
  return hipGetLastError();
}

template <int J, int MODE>
hipError_t col_launch_j(const ColArgs& a, const float2* X, float2* W, const PairRes& r, float2* Xo, hipStream_t s) {
  constexpr bool few_cells = J == 8 && MODE == COL_FWD;   // five cells' eight weights each spill 30 registers
  int spt = 0, mb = 0;
  const int nt = col_threads(a, few_cells, &spt, &mb);
  if (nt == 0) return hipErrorInvalidConfiguration;
#define COL_T(CN, SPT, MB) col_launch_t<J, MODE, CN, SPT, MB>(a, X, W, r, Xo, nt, s)
  if (spt == 2) {
    switch (a.Nz) {
      case 512: return COL_T(512, 2, 1);
      case 1024: return COL_T(1024, 2, 1);
      default: return COL_T(0, 2, 1);
    }
  }
  switch (nt <= 512 ? a.Nz : 0) {
    case 512: return COL_T(512, 5, 2);
    case 1024: return COL_T(1024, 5, 2);
    case 2048: return COL_T(2048, 5, 1);
    default: break;
  }
  if constexpr (few_cells) return COL_T(0, 3, 2);
  else return spt == 3 ? COL_T(0, 3, 2) : COL_T(0, 5, 2);
#undef COL_T
}

template <int MODE>
hipError_t col_launch(const ColArgs& a, const float2* X, float2* W, const PairRes& r, float2* Xo, hipStream_t s) {
  switch (a.J) {
    case 4: return col_launch_j<4, MODE>(a, X, W, r, Xo, s);
    case 6: return col_launch_j<6, MODE>(a, X, W, r, Xo, s);
    default: return col_launch_j<8, MODE>(a, X, W, r, Xo, s);
  }
}

}  // namespace

size_t col_lds_bytes(int N) { return (size_t)2 * col_row_cells(N) * sizeof(float4); }

int col_row_cells(int N) { return std::max(N + COL_PADK, N + N / 16 + 1); }

bool col_plan(int N, ColPlan* f, ColPlan* i, std::vector<float2>* tw) {
  for (int ns = 2; ns <= 4; ++ns) {
    int r[4];
    if (!plan_radices(N, ns, r)) continue;
    fill_plan(N, ns, r, f, tw);
    std::reverse(r, r + ns);
    fill_plan(N, ns, r, i, tw);
    return true;
  }
  return false;
}

// Threads per pair, base cells per thread and butterflies per thread.  Five
// cells share ten-cell windows between five samples (J = 6); with two butterflies
// per thread the stages that run in place take no more threads than the cells do,
// and more pairs share a CU (2048: one, whose 512 threads the cells take anyway).
// Launches of at most eight waves a CU, where a pair's chain is what counts, take
// two cells and one butterfly (forward of 245 x 600, 301 pairs: 22.2 us a call
// against 24.4).
//
// A CU holds 16 waves of these kernels, and a workgroup's waves go to its four
// SIMDs in turn, so one of five waves takes the room of eight (1400 x 1120: 561
// pairs in two rounds of 512).  Where three cells per thread fill more of it
// than five they are taken (with the natural layout, both directions of 1400 x
// 1120 50 -> 39 us), and where every pair has a CU to itself, for the shorter
// chain (2240 x 36: both directions 22.8 -> 19.3 us, forward 11.9 -> 11.4).  The
// compiled lengths have the five-cell variant only.
// few_cells: three rather than five in any case (the forward of J = 8: 128 x 512 x
// 4 items 21.7 -> 19.5 us, 1920 x 400 37.0 -> 31.8; the adjoint's registers suffice
// and five are better, 1600 x 1024 x 4 items 108 us against 129).
int col_threads(const ColArgs& a, bool few_cells, int* spt, int* mb) {
  int items = 0;
  for (int s = 1; s < a.f.ns; ++s) items = std::max(items, 4 * (a.Nz / a.f.radix[s]));
  const int64_t pairs = (int64_t)a.n_pairs * a.batch;
  auto threads = [&](int c, int m) {
    return (std::max((items + m - 1) / m, (a.span + a.J - 1 + c - 1) / c) + 63) & ~63;
  };
  *mb = 1;
  *spt = 2;
  int nt = threads(2, 1);
  if (nt <= 1024 && pairs * (nt / 64) <= 8 * 256) return nt;
  *mb = a.Nz == 2048 ? 1 : 2;
  *spt = 5;
  nt = threads(5, *mb);
  const bool compiled = a.Nz == 512 || a.Nz == 1024 || a.Nz == 2048;
  if (!compiled || (few_cells && nt > 512)) {
    auto resident = [](int t) { return t > 1024 ? 0 : 16 / ((t / 64 + 3) & ~3) * (t / 64); };
    if (few_cells || (pairs <= 256 && threads(3, 2) <= 1024) || resident(threads(3, 2)) > resident(nt)) {
      *mb = 2;
      *spt = 3;
      nt = threads(3, 2);
    }
  }
  return nt <= 1024 ? nt : 0;
}

// Whether no two samples of a column have the same base cell.  For h well above
// one cell they cannot.  At h = 1 (the default pitch) a column's t_m falls short
// of t_0 + h m by delta, which shrinks along m by delta / t a sample: where the
// boundary lies g below the fraction of t_0 + h m (modulo 1), a column passes it
// with delta = g, or g + 1, ..., and the two samples beside it stay apart if that
// drift exceeds the rounding of t (7e-10: col_sqrt at t < 32000, checked at plan
// creation).  So g must not be small, nor within rounding of 1: COL_EPS - 1e-5
// (3.5e-9 a sample, less the 1e-9 that h may lack) to 1 - 1e-6.  Other fractions
// (about 1.2e-4 of them) leave the columns to the pair kernels, which look for
// equal base cells.
static bool col_cells_distinct(const ColArgs& a) {
  const double h = 2.0 * a.ct * a.dk;
  if (h < 1.0 - 1e-9) return false;
  if (h > 1.0 + 1e-8) return true;
  const double t0 = 2.0 * a.ct * a.k_min, phi = t0 - std::floor(t0), end = phi + (h - 1.0) * (a.Mk - 1);
  const double lo = std::min(phi, end), hi = std::max(phi, end);
  for (int c = -1; c <= 1; ++c)   // the fractions with a small g, or one close to 1
    if (hi > c - COL_EPS - 1e-6 && lo < c - 1e-5) return false;
  return true;
}

// K = 2 N with a transform plan, distinct base cells, and a column's span
// within the grid
bool col_supported(const ColArgs& a) {
  int spt = 0, mb = 0;
  return a.f.ns > 0 && col_cells_distinct(a) &&
         a.span + a.J - 1 <= 2 * a.Nz && col_lds_bytes(a.Nz) <= 150 * 1024 && col_threads(a, a.J == 8, &spt, &mb) > 0;
}

hipError_t launch_col_fwd(const ColArgs& a, const float2* X1, float2* Wh, hipStream_t s) {
  return col_launch<COL_FWD>(a, X1, Wh, PairRes{}, nullptr, s);
}

hipError_t launch_col_adj(const ColArgs& a, const float2* Rh, float2* X, hipStream_t s) {
  return col_launch<COL_ADJ>(a, nullptr, const_cast<float2*>(Rh), PairRes{}, X, s);
}

hipError_t launch_col_normal(const ColArgs& a, const float2* X1, const float2* yh, double* partial, float2* X,
                             hipStream_t s) {
  PairRes r{};
  r.yh = yh;
  r.partial = partial;
  r.inv_nlat = 1.f / (float)a.nlat;
  r.nlat = (double)a.nlat;
  return col_launch<COL_NORMAL>(a, X1, nullptr, r, X, s);
}
