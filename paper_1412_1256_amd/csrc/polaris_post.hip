// Post-integration reductions on integrated spectra: channel averaging with flags (Sec. 4), the smoothed
// bandpass and the bandpass variation (Sec. 3.3.2), band moments and the Allan variances of Eq. 3 / Eq. 4
// (Sec. 3.3.1, 3.3.3).  These run once per integration or per series on data of a few MB, so they are
// latency-bound; sums are FP64 in a fixed order (run-to-run identical results).
#include "polaris_post.h"

#include "polaris_device.h"

#include <math.h>

#include <mutex>

namespace ps {

namespace {

constexpr int kNT = 256;  // threads per workgroup

typedef float f4 __attribute__((ext_vector_type(4)));

// Sum of v over the workgroup in a fixed order: wave butterflies, then wave partials in order.  Every thread
// gets the result.  sh: kNT / 64 doubles of LDS.
__device__ __forceinline__ double block_sum(double v, double* sh) {
#pragma unroll
  for (int o = 32; o > 0; o >>= 1) v += __shfl_xor(v, o, 64);
  __syncthreads();  // earlier readers of sh are done
  if ((threadIdx.x & 63) == 0) sh[threadIdx.x >> 6] = v;
  __syncthreads();
  double r = 0.0;
#pragma unroll
  for (int w = 0; w < kNT / 64; ++w) r += sh[w];
  return r;
}

// Sums over the wave of V = 2, 4, 8 or 16 values at once: at each of log2 V halving steps (lane distance 32, 16, ...) a
// lane gives away half of its values and adds its partner's other half, then butterfly steps; lane l ends with the
// sum of value l / (64 / V) in g[0] (for sixteen values 17 exchanges; each value's order of additions does not depend on V).
template <int V, int HALF = V / 2>
__device__ __forceinline__ void wave_sums(double (&g)[V], const int lane) {
  constexpr int DIST = HALF * 64 / V;
  const bool up = (lane & DIST) != 0;
#pragma unroll
  for (int i = 0; i < HALF; ++i) {
    const double give = up ? g[i] : g[i + HALF], keep = up ? g[i + HALF] : g[i];
    g[i] = keep + __shfl_xor(give, DIST, 64);
  }
  if constexpr (HALF > 1) {
    wave_sums<V, HALF / 2>(g, lane);
  } else {
#pragma unroll
    for (int o = 32 / V; o > 0; o >>= 1) g[0] += __shfl_xor(g[0], o, 64);
  }
}

__device__ __forceinline__ bool finite(double v) { return isfinite(v); }

// ------------------------------------------------------------------------------------------------
// channel averaging: bins of `factor` channels, flagged and non-finite channels left out

// factor < 64: a workgroup stages the span of nb = kSpan / factor whole bins of one spectrum in LDS (coalesced
// loads) and one thread sums each bin in channel order (a wave per bin was slower there: at factor 32 with 30
// spectra of 131072 channels 9.3 against 5.7 us).
constexpr int kSpan = 2048;

__global__ void __launch_bounds__(kNT) k_chan_avg_span(ChanAvgArgs a) {
  __shared__ float v[kSpan];
  __shared__ uint8_t ok[kSpan];
  const int64_t s = blockIdx.y;
  const int F = a.factor;
  const int nb = kSpan / F;
  const int64_t n_bins = a.n_chan / F;
  const int64_t b0 = (int64_t)blockIdx.x * nb;
  const int nbl = (int)((n_bins - b0) < nb ? (n_bins - b0) : nb);
  const int span = nbl * F;
  const float* row = a.in + s * a.n_chan + b0 * F;
  for (int i = (int)threadIdx.x; i < span; i += kNT) {
    const float x = row[i];
    const bool use = isfinite(x) && !(a.flags && a.flags[b0 * F + i]);
    v[i] = use ? x : 0.0f;
    ok[i] = use ? 1 : 0;
  }
  __syncthreads();
  for (int b = (int)threadIdx.x; b < nbl; b += kNT) {
    double sum = 0.0;
    int n = 0;
    for (int i = 0; i < F; ++i) {
      sum += (double)v[b * F + i];
      n += ok[b * F + i];
    }
    const int64_t o = s * n_bins + b0 + b;
    a.out[o] = n ? (float)(sum / n) : NAN;
    if (a.counts) a.counts[o] = n;
  }
}

// 64 <= factor <= kSpan: a wave per NB bins, straight from memory: lane j adds the channels j, j + 64, ... of a bin in order
// and the 64 lane sums are added by a fixed butterfly.  Four loads go out together, of NB bins, so that short bins keep as
// many on their way as long ones.  Bound by the read of the spectra: 30 spectra of 131072 channels at factor 256 in
// 8.2 us, 1.9 TB/s (11.2 us staged in LDS first, with a barrier between the read and the sums); 300 spectra at factor 64
// 76 us with four bins, 137 us with one, at 100 57 us with two, 89 with one.
template <int NB>
__global__ void __launch_bounds__(kNT) k_chan_avg_wave(ChanAvgArgs a) {
  constexpr int R = 4 / NB;  // loads of a bin that go out together
  const int64_t s = blockIdx.y;
  const int F = a.factor, lane = (int)threadIdx.x % 64;
  const int64_t n_bins = a.n_chan / F;
  const int64_t b = ((int64_t)blockIdx.x * (kNT / 64) + threadIdx.x / 64) * NB;  // the same for a whole wave
  if (b >= n_bins) return;
  const float* row = a.in + s * a.n_chan + b * F;
  const uint8_t* flags = a.flags ? a.flags + b * F : nullptr;
  const int bins = n_bins - b < NB ? (int)(n_bins - b) : NB;
  double sum[NB];
  int n[NB];
#pragma unroll
  for (int k = 0; k < NB; ++k) sum[k] = n[k] = 0;
  for (int i0 = 0; i0 < F; i0 += 64 * R) {
    float x[NB][R];
    bool use[NB][R];
#pragma unroll
    for (int k = 0; k < NB; ++k)
#pragma unroll
      for (int j = 0; j < R; ++j) {
        const int i = i0 + lane + 64 * j;
        const bool in = i < F && k < bins;
        x[k][j] = in ? row[k * F + i] : NAN;
        use[k][j] = !(flags && in && flags[k * F + i]);
      }
#pragma unroll
    for (int k = 0; k < NB; ++k)
#pragma unroll
      for (int j = 0; j < R; ++j) {
        const bool on = use[k][j] && isfinite(x[k][j]);
        sum[k] += on ? (double)x[k][j] : 0.0;
        n[k] += __popcll(__ballot(on));
      }
  }
#pragma unroll
  for (int k = 0; k < NB; ++k) {
#pragma unroll
    for (int o = 32; o > 0; o >>= 1) sum[k] += __shfl_xor(sum[k], o, 64);
    if (lane == 0 && k < bins) {
      a.out[s * n_bins + b + k] = n[k] ? (float)(sum[k] / n[k]) : NAN;
      if (a.counts) a.counts[s * n_bins + b + k] = n[k];
    }
  }
}

template <int NB>
static void launch_avg_wave(const ChanAvgArgs& a, int64_t n_bins, hipStream_t s) {
  constexpr int per = kNT / 64 * NB;
  hipLaunchKernelGGL(k_chan_avg_wave<NB>, dim3((unsigned)((n_bins + per - 1) / per), (unsigned)a.n_spec), dim3(kNT), 0, s, a);
}

// factor > kSpan: one workgroup per (spectrum, bin)
__global__ void __launch_bounds__(kNT) k_chan_avg_wide(ChanAvgArgs a) {
  __shared__ double sh[kNT / 64];
  const int64_t s = blockIdx.y, b = blockIdx.x;
  const int64_t n_bins = a.n_chan / a.factor;
  const int64_t c0 = b * a.factor;
  double sum = 0.0, n = 0.0;
  for (int64_t i = threadIdx.x; i < a.factor; i += kNT) {
    const float x = a.in[s * a.n_chan + c0 + i];
    if (isfinite(x) && !(a.flags && a.flags[c0 + i])) {
      sum += (double)x;
      n += 1.0;
    }
  }
  sum = block_sum(sum, sh);
  n = block_sum(n, sh);
  if (threadIdx.x == 0) {
    a.out[s * n_bins + b] = n > 0.0 ? (float)(sum / n) : NAN;
    if (a.counts) a.counts[s * n_bins + b] = (int32_t)n;
  }
}

// ------------------------------------------------------------------------------------------------
// smoothed bandpass: least-squares cubic spline, uniform knots every K channels from c0

// the four uniform cubic B-spline pieces at local position u of an interval
__device__ __forceinline__ void bspline4(double u, double (&b)[4]) {
  const double u2 = u * u, u3 = u2 * u, v = 1.0 - u;
  b[0] = v * v * v / 6.0;
  b[1] = (3.0 * u3 - 6.0 * u2 + 4.0) / 6.0;
  b[2] = (-3.0 * u3 + 3.0 * u2 + 3.0 * u + 1.0) / 6.0;
  b[3] = u3 / 6.0;
}

// W waves per knot interval j: the interval's contributions to the normal equations, Gram entries G[q][p]
// (q <= p, ten of them) of basis functions j + q, j + p and right-hand sides r[q].  Lane l of the interval's 64 W adds the
// channels l, l + 64 W, ... in order; the fourteen sums are then added over a wave's lanes together (17 exchanges, where
// fourteen whole-workgroup sums took 84 and 28 barriers) and over the waves in order.  Bound by latency, of the lanes'
// chains for wide intervals: see the launcher for W.  832 intervals of 128 channels in 3.8 us (11.1 us with fourteen
// workgroup sums per interval).
template <int W>
__global__ void __launch_bounds__(W == 1 ? kNT : 64 * W) k_spline_gram(SplineArgs a) {
  __shared__ double sh[14][W];
  const int lane = (int)threadIdx.x % 64, wave = (int)threadIdx.x / 64;
  const int64_t j = W == 1 ? (int64_t)blockIdx.x * (kNT / 64) + wave : (int64_t)blockIdx.x;  // the same for a whole wave
  if (j >= a.n_int) return;
  const int64_t lo = a.c0 + j * a.K;
  const int64_t hi = (lo + a.K) < a.c1 ? (lo + a.K) : a.c1;
  double g[16];  // fourteen sums and two zeros
#pragma unroll
  for (int q = 0; q < 16; ++q) g[q] = 0.0;
  for (int64_t c = lo + (W == 1 ? lane : (int)threadIdx.x); c < hi; c += 64 * W) {
    double b[4];
    bspline4((double)(c - lo) / (double)a.K, b);
    const double h = (double)a.h[c];
    int e = 0;
#pragma unroll
    for (int q = 0; q < 4; ++q)
#pragma unroll
      for (int p = q; p < 4; ++p) g[e++] += b[q] * b[p];
#pragma unroll
    for (int q = 0; q < 4; ++q) g[10 + q] += b[q] * h;
  }
  wave_sums<16>(g, lane);  // lane l holds value l / 4
  if constexpr (W == 1) {
    if (lane % 4 == 0 && lane / 4 < 14) a.partial[j * 14 + lane / 4] = g[0];
  } else {
    if (lane % 4 == 0 && lane / 4 < 14) sh[lane / 4][wave] = g[0];
    __syncthreads();
    if (threadIdx.x < 14) {
      double v = 0.0;
#pragma unroll
      for (int k = 0; k < W; ++k) v += sh[threadIdx.x][k];
      a.partial[j * 14 + threadIdx.x] = v;
    }
  }
}

// index of G[q][p] (q <= p) in an interval's ten Gram entries
__device__ __forceinline__ int gidx(int q, int p) {
  constexpr int start[4] = {0, 4, 7, 9};
  return start[q] + (p - q);
}

// Symmetric 3 x 3 matrices are held as (00, 10, 11, 20, 21, 22).
__device__ __forceinline__ void sym3_inverse(const double (&d)[6], double (&v)[6]) {
  const double c00 = d[2] * d[5] - d[4] * d[4], c10 = d[4] * d[3] - d[1] * d[5], c20 = d[1] * d[4] - d[2] * d[3];
  const double inv = 1.0 / (d[0] * c00 + d[1] * c10 + d[3] * c20);
  v[0] = c00 * inv;
  v[1] = c10 * inv;
  v[2] = (d[0] * d[5] - d[3] * d[3]) * inv;
  v[3] = c20 * inv;
  v[4] = (d[1] * d[3] - d[0] * d[4]) * inv;
  v[5] = (d[0] * d[2] - d[1] * d[1]) * inv;
}
__device__ __forceinline__ double sym3(const double (&d)[6], int r, int c) {
  return r >= c ? d[r * (r + 1) / 2 + c] : d[c * (c + 1) / 2 + r];
}

// One workgroup solves the normal equations.  The matrix has three entries each side of its diagonal, so in
// blocks of three rows it is block tridiagonal and symmetric; thread b holds block row b: the coupling Lb to the
// block s places before it, the diagonal block Db and the right-hand side rb.  Cyclic reduction of all rows at
// once: at distance s = 1, 2, 4, ... every row eliminates its two neighbours,
//   P = L_b D_(b-s)^-1, Q = L_(b+s)^T D_(b+s)^-1,
//   D_b -= P L_b^T + Q L_(b+s),  r_b -= P r_(b-s) + Q r_(b+s),  L_b = -P L_(b-s),
// after which it couples to the rows 2 s away; once s reaches the number of rows, a_b = D_b^-1 r_b.  The D are
// Schur complements of a positive definite matrix, so the elimination needs no pivoting, as Cholesky.
// Bound by the latency of its ~log2(n / 3) steps: 905 coefficients in 15.8 us (338 us
// as a banded Cholesky by one thread, which waits on a chain of a square root, a division and some twenty
// operations for each of the n rows).
__global__ void __launch_bounds__(kMaxSplineCoef / 3) k_spline_solve(SplineArgs a) {
  constexpr int MB = (int)(kMaxSplineCoef / 3);
  __shared__ double ls[9 * MB], dinv[6 * MB], rs[3 * MB];  // [entry][block]
  const int nb = (int)((a.n_coef + 2) / 3), b = (int)threadIdx.x;
  double L[9], D[6], r[3];
#pragma unroll
  for (int k = 0; k < 9; ++k) L[k] = 0.0;
#pragma unroll
  for (int k = 0; k < 6; ++k) D[k] = 0.0;
#pragma unroll
  for (int m = 0; m < 3; ++m) {
    const int64_t i = 3 * (int64_t)b + m;
    double row[4] = {0.0, 0.0, 0.0, 1.0}, rhs = 0.0;  // A(i, i - 3 .. i); rows past the last are the identity's
    if (i < a.n_coef) {
      row[3] = 0.0;
      // intervals j = i - 3 .. i touch basis function i (as j + q, q = i - j)
#pragma unroll
      for (int q = 0; q < 4; ++q) {
        const int64_t j = i - q;
        if (j < 0 || j >= a.n_int) continue;
        const double* G = a.partial + j * 14;
        rhs += G[10 + q];
#pragma unroll
        for (int p = 0; p <= q; ++p) row[3 - (q - p)] += G[gidx(p, q)];  // A(i, j + p), j + p = i - (q - p)
      }
    }
    r[m] = rhs;
#pragma unroll
    for (int d = 0; d <= 3; ++d) {  // column i - d: of this block for d <= m, else of the one before
      if (d <= m) D[m * (m + 1) / 2 + m - d] = row[3 - d];
      else L[3 * m + 3 + m - d] = row[3 - d];
    }
  }
  for (int s = 1; s < nb; s *= 2) {
    double v[6];
    sym3_inverse(D, v);
    __syncthreads();  // the previous step's readers are done
    if (b < nb) {
#pragma unroll
      for (int k = 0; k < 9; ++k) ls[k * MB + b] = L[k];
#pragma unroll
      for (int k = 0; k < 6; ++k) dinv[k * MB + b] = v[k];
#pragma unroll
      for (int k = 0; k < 3; ++k) rs[k * MB + b] = r[k];
    }
    __syncthreads();
    double Ln[9];
#pragma unroll
    for (int k = 0; k < 9; ++k) Ln[k] = 0.0;
    if (b < nb && b >= s) {
      double w[6], P[9];
#pragma unroll
      for (int k = 0; k < 6; ++k) w[k] = dinv[k * MB + b - s];
#pragma unroll
      for (int i = 0; i < 3; ++i)
#pragma unroll
        for (int j = 0; j < 3; ++j)
          P[3 * i + j] = L[3 * i] * sym3(w, 0, j) + L[3 * i + 1] * sym3(w, 1, j) + L[3 * i + 2] * sym3(w, 2, j);
#pragma unroll
      for (int i = 0; i < 3; ++i) {
#pragma unroll
        for (int j = 0; j <= i; ++j)
#pragma unroll
          for (int k = 0; k < 3; ++k) D[i * (i + 1) / 2 + j] -= P[3 * i + k] * L[3 * j + k];
#pragma unroll
        for (int k = 0; k < 3; ++k) r[i] -= P[3 * i + k] * rs[k * MB + b - s];
      }
#pragma unroll
      for (int k = 0; k < 3; ++k)
#pragma unroll
        for (int j = 0; j < 3; ++j) {
          const double l = ls[(3 * k + j) * MB + b - s];
#pragma unroll
          for (int i = 0; i < 3; ++i) Ln[3 * i + j] -= P[3 * i + k] * l;
        }
    }
    if (b + s < nb) {
      double w[6], l[9];
#pragma unroll
      for (int k = 0; k < 6; ++k) w[k] = dinv[k * MB + b + s];
#pragma unroll
      for (int k = 0; k < 9; ++k) l[k] = ls[k * MB + b + s];
#pragma unroll
      for (int i = 0; i < 3; ++i) {
        double Q[3];
#pragma unroll
        for (int j = 0; j < 3; ++j) Q[j] = l[i] * sym3(w, 0, j) + l[3 + i] * sym3(w, 1, j) + l[6 + i] * sym3(w, 2, j);
#pragma unroll
        for (int j = 0; j <= i; ++j)
#pragma unroll
          for (int k = 0; k < 3; ++k) D[i * (i + 1) / 2 + j] -= Q[k] * l[3 * k + j];
#pragma unroll
        for (int k = 0; k < 3; ++k) r[i] -= Q[k] * rs[k * MB + b + s];
      }
    }
#pragma unroll
    for (int k = 0; k < 9; ++k) L[k] = Ln[k];
  }
  if (b >= nb) return;
  double v[6];
  sym3_inverse(D, v);
#pragma unroll
  for (int m = 0; m < 3; ++m)
    if (3 * (int64_t)b + m < a.n_coef) a.coef[3 * b + m] = sym3(v, m, 0) * r[0] + sym3(v, m, 1) * r[1] + sym3(v, m, 2) * r[2];
}

__global__ void __launch_bounds__(kNT) k_spline_eval(SplineArgs a) {
  const int64_t c = (int64_t)blockIdx.x * kNT + threadIdx.x;
  if (c >= a.n_chan) return;
  if (c < a.c0 || c >= a.c1) {
    a.smooth[c] = NAN;
    return;
  }
  const int64_t j = (c - a.c0) / a.K;
  double b[4];
  bspline4((double)(c - a.c0 - j * a.K) / (double)a.K, b);
  double v = 0.0;
#pragma unroll
  for (int q = 0; q < 4; ++q) v += a.coef[j + q] * b[q];
  a.smooth[c] = (float)v;
}

// ------------------------------------------------------------------------------------------------

__global__ void __launch_bounds__(kNT) k_bandpass_correct(const float* __restrict__ hk, int64_t n_chan,
                                                          const float* __restrict__ smooth,
                                                          const double* __restrict__ gain,
                                                          float* __restrict__ out) {
  const int64_t s = blockIdx.y;
  const int64_t c = (int64_t)blockIdx.x * kNT + threadIdx.x;
  if (c >= n_chan) return;
  const double g = gain ? gain[s] : 1.0;
  out[s * n_chan + c] = (float)((double)hk[s * n_chan + c] / (g * (double)smooth[c]));
}

// The same with four channels per thread (16-byte loads and stores): rows of whole, 16-byte aligned quadruples.
// Bound by memory: 30 spectra of 131072 channels in 8.8 us, 3.6 TB/s (10.7 us with one channel per thread).
__global__ void __launch_bounds__(kNT) k_bandpass_correct4(const float* __restrict__ hk, int64_t n_chan,
                                                           const float* __restrict__ smooth,
                                                           const double* __restrict__ gain, float* __restrict__ out) {
  const int64_t s = blockIdx.y;
  const int64_t c = 4 * ((int64_t)blockIdx.x * kNT + threadIdx.x);
  if (c >= n_chan) return;
  const double g = gain ? gain[s] : 1.0;
  const float4 h = *reinterpret_cast<const float4*>(hk + s * n_chan + c);
  const float4 m = *reinterpret_cast<const float4*>(smooth + c);
  *reinterpret_cast<float4*>(out + s * n_chan + c) =
      make_float4((float)((double)h.x / (g * (double)m.x)), (float)((double)h.y / (g * (double)m.y)),
                  (float)((double)h.z / (g * (double)m.z)), (float)((double)h.w / (g * (double)m.w)));
}

// one workgroup per spectrum: mean of the finite channels, then the root mean square deviation from it
__global__ void __launch_bounds__(kNT) k_band_stats(const float* __restrict__ x, int64_t n_chan,
                                                    double* __restrict__ mean_sd) {
  __shared__ double sh[kNT / 64];
  const float* row = x + (int64_t)blockIdx.x * n_chan;
  double s = 0.0, n = 0.0;
  for (int64_t c = threadIdx.x; c < n_chan; c += kNT) {
    const float v = row[c];
    if (isfinite(v)) {
      s += (double)v;
      n += 1.0;
    }
  }
  s = block_sum(s, sh);
  n = block_sum(n, sh);
  const double m = n > 0.0 ? s / n : NAN;
  double q = 0.0;
  for (int64_t c = threadIdx.x; c < n_chan; c += kNT) {
    const float v = row[c];
    if (isfinite(v)) q += ((double)v - m) * ((double)v - m);
  }
  q = block_sum(q, sh);
  if (threadIdx.x == 0) {
    mean_sd[2 * blockIdx.x] = m;
    mean_sd[2 * blockIdx.x + 1] = n > 0.0 ? sqrt(q / n) : NAN;
  }
}

// Eq. 3 / Eq. 4, block form: workgroup (chunk c, series s) covers the points t of chunk c and writes, per lag
// L, the sum of squared second differences (x[t+L] - 2 x[t] + x[t-L])^2 over its t with all three samples
// finite and their count, and (normalised) the sum and count of its finite points; a second kernel adds
// the chunks of each series.  This form takes any stride and lag.
__global__ void __launch_bounds__(kNT) k_allan_part(AllanArgs a, int64_t chunks) {
  __shared__ double sh[kNT / 64];
  const int64_t s_ = blockIdx.x, c = blockIdx.y;
  const float* x = a.x + s_ * a.series_stride;
  const int64_t P = a.n_points, st = a.point_stride;
  const int64_t t0 = c * kAllanChunk, t1 = (t0 + kAllanChunk) < P ? (t0 + kAllanChunk) : P;
  double* out = a.part + (s_ * chunks + c) * (a.n_lags + 1) * 2;
  if (a.normalize) {
    double s = 0.0, n = 0.0;
    for (int64_t t = t0 + threadIdx.x; t < t1; t += kNT) {
      const float v = x[t * st];
      if (isfinite(v)) {
        s += (double)v;
        n += 1.0;
      }
    }
    s = block_sum(s, sh);
    n = block_sum(n, sh);
    if (threadIdx.x == 0) {
      out[2 * a.n_lags] = s;
      out[2 * a.n_lags + 1] = n;
    }
  }
  for (int l = 0; l < a.n_lags; ++l) {
    const int64_t L = a.lags[l];
    double s = 0.0, n = 0.0;
    const int64_t lo = t0 > L ? t0 : L, hi = t1 < P - L ? t1 : P - L;
    for (int64_t t = lo + threadIdx.x; t < hi; t += kNT) {
      const double d = (double)x[(t + L) * st] - 2.0 * (double)x[t * st] + (double)x[(t - L) * st];
      if (finite(d)) {
        s += d * d;
        n += 1.0;
      }
    }
    s = block_sum(s, sh);
    n = block_sum(n, sh);
    if (threadIdx.x == 0) {
      out[2 * l] = s;
      out[2 * l + 1] = n;
    }
  }
}

// The same partial sums for series of consecutive points (point_stride 1) whose lags are at most kWinMaxLag: the
// workgroup stages its chunk with the largest lag's points on either side in LDS (points outside the series as
// NaN) and one sweep serves NL lags.  A chunk whose staged points are all finite takes every term untested
// (its counts are known); any other tests each second difference.  Bound by FP64 issue, about ten operations a
// term, so a call of few lags has a kernel of few: 30 spectra of 131072 channels at 8 lags in 19.3 us (37.6 us reading each
// term's three points from memory, lag by lag, with a workgroup sum per lag); 300 spectra at one lag 127 us with the call
// in a sweep of eight, 57 us in one of one.  (Registers: 96 for eight lags, 44 .. 60 for fewer; one kernel that picks the
// sweep has 106 and is 5-7 % slower with eight lags.)

// Lags l0 .. l0 + NL - 1 over the n points of a chunk staged at w + lmax.
template <int NL>
__device__ __forceinline__ void allan_sweep(const AllanArgs& a, const float* __restrict__ w, const int n, const int lmax,
                                            const bool tested, const int l0, double* __restrict__ out,
                                            double (&red)[kNT / 64][2 * NL]) {
  const int tid = (int)threadIdx.x, lane = tid % 64;
  int L[NL];
  double v[2 * NL];  // sums, then counts
#pragma unroll
  for (int l = 0; l < NL; ++l) {
    L[l] = l0 + l < a.n_lags ? a.lags[l0 + l] : 0;  // 0: not a lag of this group (a zero difference)
    v[l] = v[NL + l] = 0.0;
  }
  if (!tested) {
    for (int t = tid; t < n; t += kNT) {
      const double xt = (double)w[lmax + t];
#pragma unroll
      for (int l = 0; l < NL; ++l) {
        const double d = (double)w[lmax + t + L[l]] - 2.0 * xt + (double)w[lmax + t - L[l]];
        v[l] += d * d;
      }
    }
  } else {
    for (int t = tid; t < n; t += kNT) {
      const double xt = (double)w[lmax + t];
#pragma unroll
      for (int l = 0; l < NL; ++l) {
        const double d = (double)w[lmax + t + L[l]] - 2.0 * xt + (double)w[lmax + t - L[l]];
        const bool use = finite(d);
        v[l] += use ? d * d : 0.0;
        v[NL + l] += use ? 1.0 : 0.0;
      }
    }
  }
  // the sums over the wave (lane l then holds value l / (32 / NL)), then over the waves in order
  wave_sums<2 * NL>(v, lane);
  __syncthreads();  // the previous group's readers are done
  if (lane % (32 / NL) == 0) red[tid / 64][lane / (32 / NL)] = v[0];
  __syncthreads();
  if (tid < NL && l0 + tid < a.n_lags) {
    double s = 0.0, m = 0.0;
#pragma unroll
    for (int k = 0; k < kNT / 64; ++k) {
      s += red[k][tid];
      m += red[k][NL + tid];
    }
    out[2 * (l0 + tid)] = s;
    out[2 * (l0 + tid) + 1] = tested ? m : (double)n;
  }
}

template <int NL>
__global__ void __launch_bounds__(kNT) k_allan_chunk(AllanArgs a, int64_t chunks, int lmax) {
  __shared__ float w[kAllanChunk + 2 * kWinMaxLag];
  __shared__ double red[kNT / 64][2 * NL];
  __shared__ double sh[kNT / 64];
  const int tid = (int)threadIdx.x;
  const int64_t s_ = blockIdx.x, c = blockIdx.y;
  const float* x = a.x + s_ * a.series_stride;
  const int64_t t0 = c * kAllanChunk;
  const int n = (int)((a.n_points - t0) < kAllanChunk ? (a.n_points - t0) : kAllanChunk);  // points of the chunk
  bool bad = false;
  constexpr int LD = 10;  // loads in flight per thread (two rounds at the longest lags)
  for (int i0 = tid; i0 < n + 2 * lmax; i0 += LD * kNT) {
    float v[LD];
#pragma unroll
    for (int j = 0; j < LD; ++j) {  // every load is issued, from the nearest point of the series
      const int64_t t = t0 - lmax + i0 + j * kNT;
      v[j] = x[t < 0 ? 0 : (t < a.n_points ? t : a.n_points - 1)];
    }
#pragma unroll
    for (int j = 0; j < LD; ++j) {
      const int i = i0 + j * kNT;
      const int64_t t = t0 - lmax + i;
      if (i < n + 2 * lmax) {
        const float u = t >= 0 && t < a.n_points ? v[j] : NAN;
        bad = bad || !isfinite(u);
        w[i] = u;
      }
    }
  }
  const bool tested = __syncthreads_or(bad);
  double* out = a.part + (s_ * chunks + c) * (a.n_lags + 1) * 2;
  if (a.normalize) {
    double s = 0.0, m = 0.0;
    for (int t = tid; t < n; t += kNT) {
      const float v = w[lmax + t];
      if (isfinite(v)) {
        s += (double)v;
        m += 1.0;
      }
    }
    s = block_sum(s, sh);
    m = block_sum(m, sh);
    if (tid == 0) {
      out[2 * a.n_lags] = s;
      out[2 * a.n_lags + 1] = m;
    }
  }
  for (int l0 = 0; l0 < a.n_lags; l0 += NL) allan_sweep<NL>(a, w, n, lmax, tested, l0, out, red);
}

__global__ void __launch_bounds__(kNT) k_allan_total(AllanArgs a, int64_t chunks) {
  const int64_t s_ = (int64_t)blockIdx.x * kNT + threadIdx.x;
  if (s_ >= a.n_series) return;
  const double* part = a.part + s_ * chunks * (a.n_lags + 1) * 2;
  // the chunks' (sum, count) pairs of field f added in chunk order, their loads issued eight chunks at a time
  // (one chunk at a time, each add waited for its own load)
  auto chunk_sum = [&](int f, double& s, double& n) {
    const int64_t rec = (int64_t)(a.n_lags + 1) * 2;
    const double* q = part + 2 * f;
    int64_t c = 0;
    for (; c + 8 <= chunks; c += 8) {
      double v[8][2];
#pragma unroll
      for (int j = 0; j < 8; ++j) {
        v[j][0] = q[(c + j) * rec];
        v[j][1] = q[(c + j) * rec + 1];
      }
#pragma unroll
      for (int j = 0; j < 8; ++j) {
        s += v[j][0];
        n += v[j][1];
      }
    }
    for (; c < chunks; ++c) {
      s += q[c * rec];
      n += q[c * rec + 1];
    }
  };
  double mean2 = 1.0;
  if (a.normalize) {
    double s = 0.0, n = 0.0;
    chunk_sum(a.n_lags, s, n);
    const double m = s / n;
    mean2 = m * m;
  }
  for (int l = 0; l < a.n_lags; ++l) {
    double s = 0.0, n = 0.0;
    chunk_sum(l, s, n);
    const double tau = (double)a.lags[l] * a.spacing;
    a.out[s_ * a.n_lags + l] = n > 0.0 ? s / n / (2.0 * tau * tau) / mean2 : NAN;
  }
}

// Series of kTotalChunks or more chunks: one workgroup per series, a wave per lag in turn.  Lane l adds the
// chunks l, l + 64, ... in order and the lanes' sums are added by a fixed butterfly (one thread per series walked
// the chunks of its lags one batch of loads after another: 12.7 us for 30 series of 32 chunks and 8 lags, 3.8
// here; with few chunks most lanes of a wave would have none).
constexpr int64_t kTotalChunks = 8;

__global__ void __launch_bounds__(kNT) k_allan_total_wave(AllanArgs a, int64_t chunks) {
  const int64_t s_ = blockIdx.x;
  const int lane = (int)threadIdx.x % 64;
  const int64_t rec = (int64_t)(a.n_lags + 1) * 2;
  const double* part = a.part + s_ * chunks * rec;
  auto chunk_sum = [&](int f, double& s, double& n) {
    s = n = 0.0;
    for (int64_t c = lane; c < chunks; c += 64) {
      s += part[c * rec + 2 * f];
      n += part[c * rec + 2 * f + 1];
    }
#pragma unroll
    for (int o = 32; o > 0; o >>= 1) {
      s += __shfl_xor(s, o, 64);
      n += __shfl_xor(n, o, 64);
    }
  };
  double mean2 = 1.0;
  if (a.normalize) {
    double s, n;
    chunk_sum(a.n_lags, s, n);
    const double m = s / n;
    mean2 = m * m;
  }
  for (int l = (int)threadIdx.x / 64; l < a.n_lags; l += kNT / 64) {
    double s, n;
    chunk_sum(l, s, n);
    const double tau = (double)a.lags[l] * a.spacing;
    if (lane == 0) a.out[s_ * a.n_lags + l] = n > 0.0 ? s / n / (2.0 * tau * tau) / mean2 : NAN;
  }
}

// The same for series stored side by side (series_stride 1, e.g. one series per channel of a run of
// integrations [t][channel]): a wave holds 64 consecutive series, so its loads are consecutive addresses, and
// the t range of each series is cut into kColsSlices slices handled by the workgroup's waves (one thread per
// series and slice: a single thread sweeping all t paid one memory round trip per step).  One sweep serves
// up to 8 lags (their sums in registers), so the rows t - L, t, t + L of nearby lags are reused from cache;
// each slice adds its terms in t order and the slices' sums are added in slice order (a fixed order).
constexpr int kColsSeries = 64, kColsSlices = 4;

__global__ void __launch_bounds__(kColsSeries * kColsSlices) k_allan_cols(AllanArgs a) {
  constexpr int LG = 8;
  __shared__ double red[kColsSlices][LG][2][kColsSeries];
  __shared__ double msum[kColsSlices][2][kColsSeries];
  const int lane = (int)threadIdx.x % kColsSeries, slice = (int)threadIdx.x / kColsSeries;
  const int64_t s = (int64_t)blockIdx.x * kColsSeries + lane;
  const bool valid = s < a.n_series;  // every thread still takes part in the barriers
  const float* x = a.x + (valid ? s : 0);
  const int64_t P = a.n_points, st = a.point_stride;
  const int64_t t0 = P * slice / kColsSlices, t1 = P * (slice + 1) / kColsSlices;
  double mean2 = 1.0;
  if (a.normalize) {
    double sum = 0.0, n = 0.0;
    if (valid)
      for (int64_t t = t0; t < t1; ++t) {
        const float v = x[t * st];
        if (isfinite(v)) {
          sum += (double)v;
          n += 1.0;
        }
      }
    msum[slice][0][lane] = sum;
    msum[slice][1][lane] = n;
    __syncthreads();
    double S = 0.0, N = 0.0;
#pragma unroll
    for (int k = 0; k < kColsSlices; ++k) {
      S += msum[k][0][lane];
      N += msum[k][1][lane];
    }
    const double m = S / N;
    mean2 = m * m;
  }
  for (int l0 = 0; l0 < a.n_lags; l0 += LG) {
    int64_t L[LG];
    double sum[LG], n[LG];
#pragma unroll
    for (int l = 0; l < LG; ++l) {
      L[l] = l0 + l < a.n_lags ? a.lags[l0 + l] : 0;  // 0: not a lag of this group
      sum[l] = n[l] = 0.0;
    }
    if (valid)
      for (int64_t t = t0; t < t1; ++t) {
        const double xt = (double)x[t * st];
#pragma unroll
        for (int l = 0; l < LG; ++l) {
          if (L[l] >= 1 && t >= L[l] && t < P - L[l]) {  // the same for every lane
            const double d = (double)x[(t + L[l]) * st] - 2.0 * xt + (double)x[(t - L[l]) * st];
            if (isfinite(d)) {
              sum[l] += d * d;
              n[l] += 1.0;
            }
          }
        }
      }
#pragma unroll
    for (int l = 0; l < LG; ++l) {
      red[slice][l][0][lane] = sum[l];
      red[slice][l][1][lane] = n[l];
    }
    __syncthreads();
    if (slice == 0 && valid) {
#pragma unroll
      for (int l = 0; l < LG; ++l) {
        if (l0 + l >= a.n_lags) break;
        double S = 0.0, N = 0.0;
#pragma unroll
        for (int k = 0; k < kColsSlices; ++k) {
          S += red[k][l][0][lane];
          N += red[k][l][1][lane];
        }
        const double tau = (double)L[l] * a.spacing;
        a.out[s * a.n_lags + l0 + l] = N > 0.0 && L[l] >= 1 && 2 * L[l] < P ? S / N / (2.0 * tau * tau) / mean2 : NAN;
      }
    }
    __syncthreads();  // the next lag group reuses red
  }
}

// The same for side-by-side series short enough for a workgroup to hold S of them whole in LDS, w[point][S], each
// sample read from memory once.  The second differences of a lag L are taken along runs of points L apart: thread
// (series, phase) walks t, t + L, t + 2 L, ..., so that a term needs one new sample (an LDS read and a conversion
// to FP64) beside the two it holds.  A lag has L such residues, each cut into a.runs[lag] runs of q or q + 1
// terms; the runs are dealt to the phases in rounds, consecutive phases on consecutive points.  Terms are added
// untested; a round of lags with a non-finite sum in the workgroup is taken again with each term tested.  A fixed
// order: runs of a phase in turn, phases of a wave by butterfly, waves in order.
// Bound by vector issue (per term a conversion, three FP64 operations and an address): 1800 integrations of 131072
// channels at 8 lags in 619 us, 290 us of it the read alone (3.3 TB/s in 32-byte rows); 890 us by the window form
// below, which reads and converts both outer samples of every term, with two barriers per 64 points.
template <int S, bool TEST, bool CUT>
__device__ __forceinline__ void series_lag(const float* __restrict__ w, const int P, const int L, const int m,
                                           const int s, const int ph, double& sum, double& cnt) {
  constexpr int PH = kSeriesThreads / S;
  if (L > P / 2) return;  // (2 L may exceed an int)
  const int M = P - 2 * L;  // terms
  if (M == 0) return;
  // residue r has kf terms, and one more (its last run's) when r < rem; its first e runs have q + 1 of them
  const int kf = CUT ? M / L : (M >= L ? M / L : 0), rem = M - kf * L, q = CUT ? kf / m : kf, e = CUT ? kf - q * m : 0;
  const int items = CUT ? L * m : (kf ? L : M);
  const float inv = CUT ? 1.0f / (float)L : 0.0f;
  const int step = L * S;
  for (int i0 = 0; i0 < items; i0 += PH) {
    const int i = min(i0 + ph, items - 1);  // a phase without a run repeats the last one and drops it
    int seg = 0, r = i;
    if constexpr (CUT) {  // (i + 1/2) / L is at least 1 / (2 L) from a whole number, far more than its rounding
      seg = (int)(((float)i + 0.5f) * inv);
      r = i - seg * L;
    }
    const bool more = CUT ? seg < e || (seg == m - 1 && r < rem) : r < rem;  // one term beyond q
    int at = (CUT ? r + (seg * q + min(seg, e)) * L : r) * S + s;            // the run's first sample
    double x0 = (double)w[at], x1 = (double)w[at + step];
    at += 2 * step;
    double part = 0.0, n = 0.0;
    auto add = [&](const double d) {
      if constexpr (TEST) {
        const bool use = finite(d);
        part += use ? d * d : 0.0;
        n += use ? 1.0 : 0.0;
      } else {
        part = fma(d, d, part);
      }
    };
    auto terms = [&](auto count) {
      constexpr int C = decltype(count)::value;
      float v[C];
#pragma unroll
      for (int j = 0; j < C; ++j) v[j] = w[at + j * step];
      at += C * step;
#pragma unroll
      for (int j = 0; j < C; ++j) {
        const double x2 = (double)v[j];
        add(x2 - 2.0 * x1 + x0);
        x0 = x1;
        x1 = x2;
      }
    };
    int k = q;
#pragma unroll 1
    for (; k >= 8; k -= 8) terms(std::integral_constant<int, 8>{});
    if (k & 4) terms(std::integral_constant<int, 4>{});
    if (k & 2) terms(std::integral_constant<int, 2>{});
    if (k & 1) terms(std::integral_constant<int, 1>{});
    if (CUT || i0 < rem) {  // (the same for every lane)
      const double d = (double)w[more ? at : s] - 2.0 * x1 + x0;
      if (TEST ? more : true) add(more ? d : 0.0);
    }
    const bool own = i0 + ph < items;
    sum += own ? part : 0.0;
    if constexpr (TEST) cnt += own ? n : 0.0;
  }
}

// S series to a workgroup of 512 threads, two workgroups to a CU; V: float, or four neighbouring series at once where
// rows are whole aligned quadruples.  Workgroups of 8 and 16 series share cache lines with their neighbours, which run
// on the same XCD at the same time.
template <int S, class V>
__global__ void __launch_bounds__(kSeriesThreads) k_allan_series(AllanArgs a) {
  constexpr int NT = kSeriesThreads, PH = NT / S, NW = NT / 64;
  constexpr int LG = 128 / S;  // lags per round of sums
  constexpr int W = (int)sizeof(V) / 4, G = S / W, RPS = NT / G, LD = 8;
  __shared__ double red[LG][NW][S];           // 8 KiB
  extern __shared__ __align__(16) float w[];  // [n_points][S]
  const int tid = (int)threadIdx.x, s = tid % S, ph = tid / S, lane = tid % 64, wv = tid / 64;
  const int P = (int)a.n_points;
  const int64_t sb = (int64_t)xcd_remap((int)blockIdx.x, (int)gridDim.x) * S;
  // rows in batches of LD loads, every load issued (past the end: the batch's first row again, not stored)
  const int c = W * (tid % G);
  const float* x = a.x + (sb + c < a.n_series ? sb + c : 0);
  double msum[W];
#pragma unroll
  for (int k = 0; k < W; ++k) msum[k] = 0.0;
  for (int t0 = tid / G; t0 < P; t0 += LD * RPS) {
    V d[LD];
    const float* p = x + (int64_t)t0 * a.point_stride;
#pragma unroll
    for (int j = 0; j < LD; ++j)
      d[j] = *reinterpret_cast<const V*>(p + (t0 + j * RPS < P ? (int64_t)j * RPS * a.point_stride : 0));
#pragma unroll
    for (int j = 0; j < LD; ++j)
      if (t0 + j * RPS < P) {
        *reinterpret_cast<V*>(&w[(t0 + j * RPS) * S + c]) = d[j];
#pragma unroll
        for (int k = 0; k < W; ++k) {
          if constexpr (W == 1) msum[k] += (double)d[j];
          else msum[k] += (double)d[j][k];
        }
      }
  }
  // sum over the workgroup's threads of a series, left in red[slot][wave][series]
  auto put = [&](double v, const int slot) {
#pragma unroll
    for (int o = 32; o >= S; o >>= 1) v += __shfl_xor(v, o, 64);
    if (lane < S) red[slot][wv][lane] = v;
  };
  auto total = [&](const int slot, const int c) {
    double v = 0.0;
#pragma unroll
    for (int k = 0; k < NW; ++k) v += red[slot][k][c];
    return v;
  };
  double mean2 = 1.0;  // of series tid % S
  if (a.normalize) {
#pragma unroll
    for (int k = 0; k < W; ++k) {
#pragma unroll
      for (int o = 32; o >= G; o >>= 1) msum[k] += __shfl_xor(msum[k], o, 64);
      if (lane < G) red[0][wv][c + k] = msum[k];
    }
    __syncthreads();
    double m = total(0, s), n = (double)P;
    const bool again = __syncthreads_or(!finite(m));
    if (again) {  // leave the non-finite samples out
      double v = 0.0, c = 0.0;
      for (int t = ph; t < P; t += PH) {
        const float x = w[t * S + s];
        if (isfinite(x)) {
          v += (double)x;
          c += 1.0;
        }
      }
      put(v, 0);
      put(c, 1);
      __syncthreads();
      m = total(0, s);
      n = total(1, s);
      __syncthreads();
    }
    m /= n;
    mean2 = m * m;
  }
  __syncthreads();  // the window is complete, and red free
  for (int l0 = 0; l0 < a.n_lags; l0 += LG) {
    const int nl = a.n_lags - l0 < LG ? a.n_lags - l0 : LG;
    for (int l = 0; l < nl; ++l) {
      double sum = 0.0, cnt = 0.0;
      if (a.runs[l0 + l] > 1) series_lag<S, false, true>(w, P, a.lags[l0 + l], a.runs[l0 + l], s, ph, sum, cnt);
      else series_lag<S, false, false>(w, P, a.lags[l0 + l], 1, s, ph, sum, cnt);
      put(sum, l);
    }
    __syncthreads();
    // one thread per (lag, series) of the round
    const int l = tid / S;
    const bool writer = l < nl && sb + s < a.n_series;
    auto write = [&](const double sum, const double n) {
      const double tau = (double)a.lags[l0 + l] * a.spacing;
      a.out[(sb + s) * a.n_lags + l0 + l] = n > 0.0 ? sum / n / (2.0 * tau * tau) / mean2 : NAN;
    };
    double sum = 0.0;
    if (writer) sum = total(l, s);
    const bool again = __syncthreads_or(writer && !finite(sum));
    if (!again) {
      if (writer) write(sum, (double)P - 2.0 * a.lags[l0 + l]);  // every term counts (none: a negative count)
      continue;
    }
    for (int k = 0; k < nl; ++k) {  // a lag at a time: its sums in slot 0, its counts in slot 1
      double v = 0.0, c = 0.0;
      if (a.runs[l0 + k] > 1) series_lag<S, true, true>(w, P, a.lags[l0 + k], a.runs[l0 + k], s, ph, v, c);
      else series_lag<S, true, false>(w, P, a.lags[l0 + k], 1, s, ph, v, c);
      put(v, 0);
      put(c, 1);
      __syncthreads();
      if (writer && l == k) write(total(0, s), total(1, s));
      __syncthreads();
    }
  }
}

// The same for side-by-side series whose lags are at most kWinMaxLag, through a window of the series held in
// LDS.  A workgroup owns 32 neighbouring series (128-byte rows of the [t][series] array) and walks t in steps
// of 64 rows; every row is read from memory once and then serves all its second differences from LDS.  The
// window is a ring of kWinRing rows (the rows t - 2 Lmax .. t + 63 of a step) whose first 64 slots are
// repeated after its end, so a run of 64 consecutive rows never wraps.  Thread (group g, phase q, half h)
// holds the four series 4g .. 4g+3 (16-byte LDS reads) and takes the point t = r0 - Lmax + q of every step
// r0 (the point whose t + Lmax has just arrived) for lags 4h .. 4h+3 of a group of up to eight.  A term is
// added without a finiteness test: a series with a non-finite sample ends with a non-finite sum, and only
// then is that (series, lag) summed again term by term, leaving out non-finite triples.  The 64 phases'
// sums are added in phase order.  Needs rows that are 8-byte aligned and a row stride of whole float pairs.
constexpr int kWinSeries = 32, kWinStep = 64, kWinGroups = kWinSeries / 4, kWinLags = 8, kWinAhead = 2;
constexpr int kWinHalfLags = kWinLags / 2;
constexpr int kWinRing = 2 * kWinMaxLag + 2 * kWinStep;
constexpr int kWinThreads = kWinGroups * kWinStep * 2;

__global__ void __launch_bounds__(kWinThreads) k_allan_window(AllanArgs a) {
  __shared__ __align__(16) float buf[(kWinRing + kWinStep) * kWinSeries];
  double* red = reinterpret_cast<double*>(buf);  // [lag][phase][series] phase sums, after a sweep
  __shared__ double meanv[kWinSeries];            // squared series means (normalisation)
  static_assert(kWinLags * kWinStep * kWinSeries * 8 <= (kWinRing + kWinStep) * kWinSeries * 4,
                "the phase sums fit in the ring");
  const int tid = (int)threadIdx.x;
  const int g = tid % kWinGroups, q = (tid / kWinGroups) % kWinStep;
  // the half is the same for a whole wave (512-thread halves): made visibly uniform, so the lag and ring-slot
  // arithmetic below runs on the scalar unit
  const int h = __builtin_amdgcn_readfirstlane(tid / (kWinGroups * kWinStep));
  const int64_t sb = (int64_t)blockIdx.x * kWinSeries;  // first series of the workgroup
  const int P = (int)a.n_points;                          // < 2^31 (checked by the launcher)
  const int64_t st = a.point_stride;
  // loads: row r0 + q, the two series 4g + 2h, 4g + 2h + 1 (a wave reads whole 128-byte rows).  The series
  // count is even, so a pair is wholly in or out; every load is issued (past the end: from row P - 1 or the
  // first pair, a valid address) and replaced by zeros, so no load sits behind a branch.
  const int ls = 4 * g + 2 * h;
  const bool pin = sb + ls < a.n_series;
  const float* xl = a.x + (pin ? sb + ls : 0);
  typedef float f2 __attribute__((ext_vector_type(2)));
  // (the zeros are substituted when the pair enters the ring, so the load is not waited for until then)
  auto fetch = [&](f2& d, int r) { d = *reinterpret_cast<const f2*>(xl + (int64_t)(r < P ? r : P - 1) * st); };
  auto wrap = [](int k) { return k >= kWinRing ? k - kWinRing : k; };
  // ring slot X + q of this lane: a per-lane byte offset plus the wave-uniform X times the row bytes (one
  // vector add per read)
  const uint32_t lane_b = (uint32_t)(q * kWinSeries + 4 * g) * 4u;
  auto rdq = [&](int x) {
    const uint32_t off = lane_b + (uint32_t)__builtin_amdgcn_readfirstlane(x) * (kWinSeries * 4u);
    return *reinterpret_cast<const f4*>(reinterpret_cast<const char*>(buf) + off);
  };
  double xs[2] = {0, 0}, xn[2] = {0, 0};  // finite samples of the loaded series (normalisation), first sweep
  for (int l0 = 0; l0 < a.n_lags; l0 += kWinLags) {
    int L[kWinLags];
    int lmax = 1;
#pragma unroll
    for (int l = 0; l < kWinLags; ++l) {
      L[l] = l0 + l < a.n_lags ? a.lags[l0 + l] : 0;  // 0: not a lag of this group
      lmax = L[l] > lmax ? L[l] : lmax;
    }
    int Lh[kWinHalfLags];
#pragma unroll
    for (int l = 0; l < kWinHalfLags; ++l) Lh[l] = h ? L[kWinHalfLags + l] : L[l];
    double S[kWinHalfLags][4];
#pragma unroll
    for (int l = 0; l < kWinHalfLags; ++l)
#pragma unroll
      for (int c = 0; c < 4; ++c) S[l][c] = 0.0;
    f2 pre[kWinAhead];
    // issued in step order (the loop then finds the same order each time round: a step waits only for the
    // loads issued before its own)
#pragma unroll
    for (int u = 0; u < kWinAhead; ++u) {
      fetch(pre[u], u * kWinStep + q);
      __builtin_amdgcn_sched_barrier(0);
    }
    int k0 = 0;                // slot of row r0
    int bt = kWinRing - lmax;  // slot of row r0 - lmax (lmax <= kWinMaxLag < kWinRing)
    // the point t = r0 - lmax + q of step r0 counts for lag L when L <= t < P - L: every point of the step
    // counts for every lag of this half (the same for every lane) in a contiguous middle range of steps
    auto step_all = [&](const int r0) {
      bool all = true;
#pragma unroll
      for (int l = 0; l < kWinHalfLags; ++l)
        all = all && Lh[l] >= 1 && r0 - lmax >= Lh[l] && r0 - lmax + kWinStep - 1 < P - Lh[l];
      return all;
    };
    auto step = [&](const int r0, f2& d, auto masked) {
      __syncthreads();  // every thread is done with the previous step's rows
      {
        if (!(pin && r0 + q < P)) d = f2{0.f, 0.f};
        const int k = wrap(k0 + q);
        *reinterpret_cast<f2*>(&buf[k * kWinSeries + ls]) = d;
        if (k < kWinStep) *reinterpret_cast<f2*>(&buf[(k + kWinRing) * kWinSeries + ls]) = d;
        if (l0 == 0 && a.normalize && r0 + q < P) {
          if (isfinite(d.x)) {
            xs[0] += (double)d.x;
            xn[0] += 1.0;
          }
          if (isfinite(d.y)) {
            xs[1] += (double)d.y;
            xn[1] += 1.0;
          }
        }
      }
      fetch(d, r0 + kWinAhead * kWinStep + q);
      __syncthreads();
      const int t = r0 - lmax + q;
      const f4 b = rdq(bt);
      const double xb[4] = {b.x, b.y, b.z, b.w};
#pragma unroll
      for (int l = 0; l < kWinHalfLags; ++l) {
        const f4 ua = rdq(wrap(bt + Lh[l]));
        const f4 dc = rdq(bt >= Lh[l] ? bt - Lh[l] : bt - Lh[l] + kWinRing);
        const double xa[4] = {ua.x, ua.y, ua.z, ua.w}, xc[4] = {dc.x, dc.y, dc.z, dc.w};
        const bool use = !decltype(masked)::value || (Lh[l] >= 1 && t >= Lh[l] && t < P - Lh[l]);
#pragma unroll
        for (int c = 0; c < 4; ++c) {
          const double dd = xa[c] - 2.0 * xb[c] + xc[c];
          const double e = use ? dd : 0.0;  // an exact zero term outside the lag's range
          S[l][c] = fma(e, e, S[l][c]);
        }
      }
      k0 = wrap(k0 + kWinStep);
      bt = wrap(bt + kWinStep);
    };
    // Every step of an unrolled group runs: a step past the last point writes zero rows and adds exact
    // zeros (its points are out of every lag's range), and no load then sits behind a branch, so each step
    // waits only for its own rows while the later steps' loads stay in flight.
    // Three loops over the step groups: those before the middle range, the middle range (no range test), and
    // those after it; each loop then has one definition of the sums (a test inside one loop had the compiler
    // copy all sixteen FP64 sums on every step).
    constexpr int GS = kWinAhead * kWinStep;  // rows per step group
    auto group_all = [&](const int r0) {
      bool all = true;
#pragma unroll
      for (int u = 0; u < kWinAhead; ++u) all = all && step_all(r0 + u * kWinStep);
      return all;
    };
    int r0 = 0;
    for (; r0 < P + lmax && !group_all(r0); r0 += GS) {
#pragma unroll
      for (int u = 0; u < kWinAhead; ++u) step(r0 + u * kWinStep, pre[u], std::true_type{});
    }
    for (; r0 < P + lmax && group_all(r0); r0 += GS) {
#pragma unroll
      for (int u = 0; u < kWinAhead; ++u) step(r0 + u * kWinStep, pre[u], std::false_type{});
    }
    for (; r0 < P + lmax; r0 += GS) {
#pragma unroll
      for (int u = 0; u < kWinAhead; ++u) step(r0 + u * kWinStep, pre[u], std::true_type{});
    }
    __syncthreads();  // the ring is free: it holds the phase sums from here on
    if (l0 == 0 && a.normalize) {  // series means: [2][phase][series] sums, added in phase order
#pragma unroll
      for (int c = 0; c < 2; ++c) {
        red[q * kWinSeries + ls + c] = xs[c];
        red[(kWinStep + q) * kWinSeries + ls + c] = xn[c];
      }
      __syncthreads();
      if (tid < kWinSeries) {
        double sx = 0.0, sn = 0.0;
        for (int p = 0; p < kWinStep; ++p) {
          sx += red[p * kWinSeries + tid];
          sn += red[(kWinStep + p) * kWinSeries + tid];
        }
        meanv[tid] = (sx / sn) * (sx / sn);
      }
      __syncthreads();
    }
#pragma unroll
    for (int l = 0; l < kWinHalfLags; ++l)
#pragma unroll
      for (int c = 0; c < 4; ++c) red[((h * kWinHalfLags + l) * kWinStep + q) * kWinSeries + 4 * g + c] = S[l][c];
    __syncthreads();
    // writers: one thread per (series, lag) of the group
    if (tid < kWinSeries * kWinLags) {
      const int c = tid % kWinSeries, l = tid / kWinSeries;
      const int64_t sr = sb + c;
      if (sr < a.n_series && l0 + l < a.n_lags) {
        const double mean2 = a.normalize ? meanv[c] : 1.0;
        double sum = 0.0;
        for (int p = 0; p < kWinStep; ++p) sum += red[(l * kWinStep + p) * kWinSeries + c];
        const int64_t Ll = L[l];
        double n = (double)(P - 2 * Ll > 0 ? P - 2 * Ll : 0);  // every term counts (finite sum)
        if (!isfinite(sum)) {
          // a non-finite sample in the series: the terms again, in t order, without the non-finite ones
          const float* xc = a.x + sr;
          sum = 0.0;
          n = 0.0;
          for (int64_t t = Ll; t < P - Ll; ++t) {
            const double dd = (double)xc[(t + Ll) * st] - 2.0 * (double)xc[t * st] + (double)xc[(t - Ll) * st];
            if (isfinite(dd)) {
              sum += dd * dd;
              n += 1.0;
            }
          }
        }
        const double tau = (double)Ll * a.spacing;
        a.out[sr * a.n_lags + l0 + l] = n > 0.0 && Ll >= 1 && 2 * Ll < P ? sum / n / (2.0 * tau * tau) / mean2 : NAN;
      }
    }
    __syncthreads();  // the next lag group refills the ring
  }
}

}  // namespace

hipError_t launch_channel_average(const ChanAvgArgs& a, hipStream_t s) {
  const int64_t n_bins = a.n_chan / a.factor;
  if (a.factor >= 64 && a.factor <= kSpan) {
    if (a.factor == 64) launch_avg_wave<4>(a, n_bins, s);
    else if (a.factor <= 128) launch_avg_wave<2>(a, n_bins, s);
    else launch_avg_wave<1>(a, n_bins, s);
  } else if (a.factor < 64) {
    const int nb = kSpan / a.factor;
    const dim3 grid((unsigned)((n_bins + nb - 1) / nb), (unsigned)a.n_spec);
    hipLaunchKernelGGL(k_chan_avg_span, grid, dim3(kNT), 0, s, a);
  } else {
    hipLaunchKernelGGL(k_chan_avg_wide, dim3((unsigned)n_bins, (unsigned)a.n_spec), dim3(kNT), 0, s, a);
  }
  return hipGetLastError();
}

// ---- scratch of the allocation-free bandpass fit: a file-scope device array, one copy per GPU, found once
// per device with hipGetSymbolAddress (host code may use only that address, never the array's name)
static __device__ __align__(256) unsigned char scratch[kBandpassScratchBytes];

hipError_t bandpass_scratch(hipStream_t stream, void** ptr) {
  static std::mutex mu;
  static void* addr[kMaxDevices] = {};
  int dev = -1;
  hipError_t e = stream ? hipStreamGetDevice(stream, &dev) : hipGetDevice(&dev);
  if (e != hipSuccess) return e;
  if (dev < 0 || dev >= kMaxDevices) return hipErrorInvalidDevice;
  std::lock_guard<std::mutex> lock(mu);
  if (!addr[dev]) {
    int cur = -1;
    if ((e = hipGetDevice(&cur)) != hipSuccess) return e;
    if (cur != dev && (e = hipSetDevice(dev)) != hipSuccess) return e;
    void* p = nullptr;
    e = hipGetSymbolAddress(&p, HIP_SYMBOL(scratch));
    if (cur != dev) {
      const hipError_t r = hipSetDevice(cur);
      if (e == hipSuccess) e = r;
    }
    if (e != hipSuccess) return e;
    addr[dev] = p;
  }
  *ptr = addr[dev];
  return hipSuccess;
}

hipError_t launch_bandpass_fit(const SplineArgs& a, hipStream_t s) {
  // Waves per interval: one up to 1024 channels (there the solve or, with thousands of intervals, the waves themselves
  // fill the chip: 2^21 channels 44.9 us, 46.5 with four), four beyond (2^17 channels at 4096: 27.1 -> 17.0 us) and
  // sixteen from 8192 on, where few intervals are left (16384: 73.2 us with one, 25.8 with four, 23.1 with sixteen).
  const int W = a.K > 1024 ? (a.K < 8192 ? 4 : 16) : 1;
  if (W == 1) hipLaunchKernelGGL(k_spline_gram<1>, dim3((unsigned)((a.n_int + kNT / 64 - 1) / (kNT / 64))), dim3(kNT), 0, s, a);
  else if (W == 4) hipLaunchKernelGGL(k_spline_gram<4>, dim3((unsigned)a.n_int), dim3(256), 0, s, a);
  else hipLaunchKernelGGL(k_spline_gram<16>, dim3((unsigned)a.n_int), dim3(1024), 0, s, a);
  // one thread per block of three coefficients (at most kMaxSplineCoef / 3), in whole waves
  const unsigned blocks = (unsigned)((a.n_coef + 2) / 3);
  hipLaunchKernelGGL(k_spline_solve, dim3(1), dim3((blocks + 63) / 64 * 64), 0, s, a);
  hipLaunchKernelGGL(k_spline_eval, dim3((unsigned)((a.n_chan + kNT - 1) / kNT)), dim3(kNT), 0, s, a);
  return hipGetLastError();
}

hipError_t launch_bandpass_correct(const float* hk, int64_t n_spec, int64_t n_chan, const float* smooth,
                                   const double* gain, float* out, hipStream_t s) {
  const uintptr_t at = reinterpret_cast<uintptr_t>(hk) | reinterpret_cast<uintptr_t>(smooth) | reinterpret_cast<uintptr_t>(out);
  if (n_chan % 4 == 0 && at % 16 == 0) {
    hipLaunchKernelGGL(k_bandpass_correct4, dim3((unsigned)((n_chan / 4 + kNT - 1) / kNT), (unsigned)n_spec), dim3(kNT),
                       0, s, hk, n_chan, smooth, gain, out);
    return hipGetLastError();
  }
  hipLaunchKernelGGL(k_bandpass_correct, dim3((unsigned)((n_chan + kNT - 1) / kNT), (unsigned)n_spec), dim3(kNT), 0,
                     s, hk, n_chan, smooth, gain, out);
  return hipGetLastError();
}

hipError_t launch_band_stats(const float* x, int64_t n_spec, int64_t n_chan, double* mean_sd, hipStream_t s) {
  hipLaunchKernelGGL(k_band_stats, dim3((unsigned)n_spec), dim3(kNT), 0, s, x, n_chan, mean_sd);
  return hipGetLastError();
}

// Runs per residue of lag L of the whole-series form with ph phases: cutting a residue's terms into m runs fills the
// last round of phases better, while each run costs about as much as four more terms (its two first samples, its
// bounds); the m with the least time for the rounds is taken, among those whose cut runs have an odd number of
// terms, so that the runs of neighbouring phases start on different banks.
static int series_runs(int P, int L, int ph) {  // (P at most a few thousand: whole-series form)
  if (L > P / 4) return 1;
  const int kf = (P - 2 * L) / L;
  int best = 1, cost = (L + ph - 1) / ph * (kf + 4);
  for (int m = 2; m <= kf && m <= 64; ++m) {
    const int q = kf / m;
    if (q % 2 == 0) continue;
    const int c = (L * m + ph - 1) / ph * (q + 4);
    if (c < cost) {
      cost = c;
      best = m;
    }
  }
  return best;
}

// Series per workgroup of the whole-series form (0: too long): as many as fit half a CU's LDS, up to 64, so that
// short series still make a workgroup's worth of work, but no more than leave 256 workgroups (2048 series of 100 points at
// 8 lags: 14.9 us in 32 workgroups, 12.2 in 256, the rate of the call itself), or 128 of 8 series, whose rows are a
// quarter of a cache line (4000 series of 1100 points: 18.7 us in 250 workgroups, 20.4 in 500).
static int series_per_block(int64_t P, int64_t n_series) {
  int S = 64;
  while (S > 8 && (P * S * 4 > kSeriesLdsBytes || n_series <= (S > 16 ? 255 : 127) * S)) S /= 2;
  return P * S * 4 <= kSeriesLdsBytes ? S : 0;
}

template <int S>
static void launch_series(AllanArgs a, hipStream_t s) {
  for (int l = 0; l < a.n_lags; ++l) a.runs[l] = series_runs((int)a.n_points, a.lags[l], kSeriesThreads / S);
  const dim3 grid((unsigned)((a.n_series + S - 1) / S)), block(kSeriesThreads);
  const size_t lds = (size_t)a.n_points * S * 4;
  if (reinterpret_cast<uintptr_t>(a.x) % 16 == 0 && a.point_stride % 4 == 0 && a.n_series % 4 == 0)
    hipLaunchKernelGGL((k_allan_series<S, f4>), grid, block, lds, s, a);
  else
    hipLaunchKernelGGL((k_allan_series<S, float>), grid, block, lds, s, a);
}

static bool allan_cols(int64_t n_series, int64_t point_stride, int64_t series_stride) {
  return series_stride == 1 && point_stride >= n_series && n_series >= 64;
}

int64_t allan_part_doubles(int64_t n_points, int64_t n_series, int64_t point_stride, int64_t series_stride,
                           int n_lags) {
  if (allan_cols(n_series, point_stride, series_stride)) return 0;
  const int64_t chunks = n_points > 0 ? (n_points + kAllanChunk - 1) / kAllanChunk : 1;
  return n_series * chunks * (n_lags + 1) * 2;
}

hipError_t launch_allan(const AllanArgs& a, hipStream_t s) {
  int lmax = 0;
  for (int l = 0; l < a.n_lags; ++l) lmax = a.lags[l] > lmax ? a.lags[l] : lmax;
  const bool rows16 = reinterpret_cast<uintptr_t>(a.x) % 8 == 0 && a.point_stride % 2 == 0 && a.n_series % 2 == 0;
  const bool cols = allan_cols(a.n_series, a.point_stride, a.series_stride);
  const int S = cols && a.n_points >= 1 ? series_per_block(a.n_points, a.n_series) : 0;
  if (S) {  // up to 2288 points
    switch (S) {
      case 64: launch_series<64>(a, s); break;
      case 32: launch_series<32>(a, s); break;
      case 16: launch_series<16>(a, s); break;
      default: launch_series<8>(a, s); break;
    }
  } else if (cols && lmax <= kWinMaxLag && rows16 &&
      a.n_points >= 1 && a.n_points < (int64_t(1) << 31)) {  // (no rows: the column form writes NaN)
    hipLaunchKernelGGL(k_allan_window, dim3((unsigned)((a.n_series + kWinSeries - 1) / kWinSeries)),
                       dim3(kWinThreads), 0, s, a);
  } else if (cols) {
    hipLaunchKernelGGL(k_allan_cols, dim3((unsigned)((a.n_series + kColsSeries - 1) / kColsSeries)),
                       dim3(kColsSeries * kColsSlices), 0, s, a);
  } else {
    const int64_t chunks = a.n_points > 0 ? (a.n_points + kAllanChunk - 1) / kAllanChunk : 1;
    const dim3 grid((unsigned)a.n_series, (unsigned)chunks);
    if (a.point_stride == 1 && lmax <= kWinMaxLag && a.n_points >= 1) {
      if (a.n_lags == 1) hipLaunchKernelGGL(k_allan_chunk<1>, grid, dim3(kNT), 0, s, a, chunks, lmax);
      else if (a.n_lags == 2) hipLaunchKernelGGL(k_allan_chunk<2>, grid, dim3(kNT), 0, s, a, chunks, lmax);
      else if (a.n_lags <= 4) hipLaunchKernelGGL(k_allan_chunk<4>, grid, dim3(kNT), 0, s, a, chunks, lmax);
      else hipLaunchKernelGGL(k_allan_chunk<8>, grid, dim3(kNT), 0, s, a, chunks, lmax);
    } else
      hipLaunchKernelGGL(k_allan_part, grid, dim3(kNT), 0, s, a, chunks);
    if (chunks >= kTotalChunks)
      hipLaunchKernelGGL(k_allan_total_wave, dim3((unsigned)a.n_series), dim3(kNT), 0, s, a, chunks);
    else
      hipLaunchKernelGGL(k_allan_total, dim3((unsigned)((a.n_series + kNT - 1) / kNT)), dim3(kNT), 0, s, a, chunks);
  }
  return hipGetLastError();
}

}  // namespace ps
