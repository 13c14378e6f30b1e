// Single-pass transform of short frames (N = 2^8 .. 2^12): T = N / 16 threads hold a whole frame of a pair,
// z = x + i y, 16 points each in registers, and transform it by two or three Stockham passes of radix 4, 8 or 16 with
// exchanges through LDS; the cross-power products of its channels are added to FP64 registers, and only the packed
// input is read from HBM.  A thread group is one accumulator slot of one pair: absolute frame a of the integration
// belongs to slot a mod G, and the group adds its frames in order, then writes the slot in the layout of the
// four-step row pass, so Stokes, spectra, state export and the backward read it unchanged.
#include <hip/hip_ext.h>

#include "polaris_fused.h"
#include "polaris_device.h"

namespace ps {

namespace {

// threads of a workgroup, and frames (slots) side by side in it
template <int N>
constexpr int fused_nt() {
  return N / 16 < 64 ? 64 : N / 16;
}

// Raw words of a thread's 16 time samples of a frame.  MODE 1 (two streams, the pair (0, 1)) and 2 (four streams):
// one word of a time sample's codes per point (a byte of two samples for two 2-bit streams); MODE 0: the byte (or
// float) of each stream's item.
template <int N, int BITS, int MODE>
struct FusedLoader {
  static constexpr int T = Passes16<N>::T;
  static constexpr int TB = MODE == 1 ? 2 * BITS : 4 * BITS;  // bits of a time sample's word
  uint32_t x[16], y[MODE == 0 ? 16 : 1];
  template <class P>
  __device__ __forceinline__ void fetch(const P base, const int ts, const int S, const int sx, const int sy) {
    // item places are formed anew each frame (an opaque zero keeps the compiler from holding all of them)
    int tz = ts;
    if constexpr (MODE == 0) {
      int z;
      asm volatile("v_mov_b32 %0, 0" : "=v"(z));
      tz += z;
    }
#pragma unroll
    for (int k = 0; k < 16; ++k) {
      if constexpr (MODE == 0) {
        const uint32_t it = (uint32_t)((tz + k * T) * S);
        x[k] = item(base, it + sx);
        y[k] = item(base, it + sy);
      } else {
        const P q = base + ((uint32_t)(ts * TB) >> 3) + k * T * TB / 8;
        if constexpr (TB == 32) x[k] = *(const __attribute__((address_space(1))) uint32_t*)q;
        else if constexpr (TB == 16) x[k] = *(const __attribute__((address_space(1))) uint16_t*)q;
        else x[k] = *q;
      }
    }
  }
  template <class P>
  static __device__ __forceinline__ uint32_t item(const P base, uint32_t i) {
    if constexpr (BITS == 32) return *(const __attribute__((address_space(1))) uint32_t*)(base + 4u * i);
    else return *(base + ((i * BITS) >> 3));
  }
  // the code at bit `shift` of a word, as its level (a float item: the word itself)
  static __device__ __forceinline__ float level(uint32_t w, uint32_t shift) {
    if constexpr (BITS == 32) return __uint_as_float(w);
    else if constexpr (BITS == 8) return (float)(int)(int8_t)(uint8_t)(w >> shift);
    else return (float)(2 * (int)((w >> shift) & ((1u << BITS) - 1u)) - ((1 << BITS) - 1));
  }
  __device__ __forceinline__ float2 get(const int k, const int ts, const int S, const int sx, const int sy) const {
    if constexpr (MODE == 0) {
      const uint32_t it = (uint32_t)((ts + k * T) * S) * BITS;  // (bit place; only its low three bits count)
      return BITS >= 8 ? make_float2(level(x[k], 0), level(y[k], 0))
                       : make_float2(level(x[k], (it + sx * BITS) & 7u), level(y[k], (it + sy * BITS) & 7u));
    } else {
      const uint32_t s0 = TB < 8 ? (uint32_t)(ts & 1) * TB : 0u;  // (T is even: k T does not change the half)
      const int fx = MODE == 1 ? 0 : sx, fy = MODE == 1 ? 1 : sy;
      return make_float2(level(x[k], s0 + fx * BITS), level(x[k], s0 + fy * BITS));
    }
  }
};

// Bound by vector issue and the latency of its exchanges at two waves per SIMD (some 930 vector instructions per 16
// points of 64 lanes, three quarters of them the transform; LDS active a quarter of the time).  4096 frames of 4096
// points, two int8 streams: 40.7 us, 84.3 us with 8 points per thread, byte loads, the input staged through LDS and
// two barriers per pass.  N / 16 threads per frame leave room for the twiddles, the window and the eight channels'
// sums in registers (240); every pass of radix 16 saves an exchange against three of radix 8.
template <int N, int BITS, int MODE>
__global__ void __launch_bounds__(fused_nt<N>()) k_fused(FusedArgs a) {
  using F = Passes16<N>;
  constexpr int T = F::T, SPW = fused_nt<N>() / T, R0 = F::R0, R1 = F::R1;
  // frames of several waves: two buffers, so that three barriers per frame suffice (see the frame loop)
  constexpr int NBUF = F::WAVE ? 1 : 2;
  __shared__ __align__(16) float2 buf[SPW][NBUF][F::LEN];
  const int sub = SPW > 1 ? (int)threadIdx.x / T : 0, ts = SPW > 1 ? (int)threadIdx.x % T : (int)threadIdx.x;
  const int g = (int)blockIdx.x * SPW + sub, p = (int)blockIdx.y;
  const int sx = a.px[p], sy = a.py[p];
  // this slot's frames of the launch: f = f_first + j G (absolute frame F0 + f = g mod G)
  const int f_first = (int)(((int64_t)g - a.F0 % a.G + a.G) % a.G);
  const int n_loc = g < a.G && f_first < a.n_frames ? (a.n_frames - f_first + a.G - 1) / a.G : 0;
  if (SPW == 1 && n_loc == 0) return;
  // slots that share a wave differ by at most one frame: all run the longest count, the others' extra frame is dropped
  const int n_run = SPW == 1 ? n_loc : (a.n_frames + a.G - 1) / a.G;
  const bool prior = a.F0 > g;  // the slot already holds frames of this integration
  double* slot = a.acc + (int64_t)g * a.slot_stride;

  float2 w1[R1 ? R1 - 1 : 1], w2[15];
#pragma unroll
  for (int r = 1; r < (R1 ? R1 : 1); ++r) w1[r - 1] = a.tw[r * (ts & (R0 - 1)) * (N / (R0 * (R1 ? R1 : 1)))];
#pragma unroll
  for (int r = 1; r < 16; ++r) w2[r - 1] = a.tw[r * ts];
  float win[16];
#pragma unroll
  for (int k = 0; k < 16; ++k) win[k] = a.win[ts + k * T];

  // channels ts + r T, r < 8: channel k = k1 + N1 k2 (k1 < N1, k2 < N2/2) sits in unit u of row half `half` (the
  // row pass's layout)
  const int U = a.N1 / 2, L = a.N2;
  auto place = [&](const int k) {
    const int k1 = k & (a.N1 - 1), k2 = k / a.N1;
    int u, half;
    if (k1 == 0) { u = 0; half = 0; }
    else if (2 * k1 == a.N1) { u = 0; half = 1; }
    else if (2 * k1 < a.N1) { u = k1; half = 0; }
    else { u = a.N1 - k1; half = 1; }
    return (p * U + u) * 4 * L + half * (L / 2) + k2;
  };
  double sum[4][8];
#pragma unroll
  for (int r = 0; r < 8; ++r) {
    const int at = place(ts + r * T);
#pragma unroll
    for (int q = 0; q < 4; ++q) sum[q][r] = prior && n_loc ? slot[at + q * L] : 0.0;
  }

  using G1 = const __attribute__((address_space(1))) uint8_t*;
  auto frame_base = [&](int j) {  // frame f_first + j G of the launch
    const int f = SPW == 1 ? f_first + j * a.G : min(f_first + j * a.G, a.n_frames - 1);
    const uint8_t* q = a.in + (int64_t)f * a.hop * a.S * BITS / 8;
    if constexpr (SPW == 1) return uniform_gptr(q);
    else return (G1)(uintptr_t)q;
  };
  FusedLoader<N, BITS, MODE> ld;
  ld.fetch(frame_base(0), ts, a.S, sx, sy);
  for (int j = 0; j < n_run; ++j) {
    float2* const b0 = buf[sub][NBUF == 2 ? (j & 1) : 0];
    float2* const b1 = buf[sub][NBUF == 2 ? 1 - (j & 1) : 0];
    float2 v[16];
#pragma unroll
    for (int k = 0; k < 16; ++k) {
      const float2 c = ld.get(k, ts, a.S, sx, sy);
      v[k] = make_float2(c.x * win[k], c.y * win[k]);
    }
    // the next frame's words, in flight through this frame (the last frame reads itself again)
    ld.fetch(frame_base(j + 1 < n_run ? j + 1 : j), ts, a.S, sx, sy);
    // Buffers of frames of several waves: the first exchange uses b0, the second b1 and the mirror b0 again, and the
    // next frame the other way round, so that a buffer's readers have always passed a barrier before it is written.
    dft16<R0, false>(v, w2);
    exchange16<N, R0, 1>(v, ts, b0);
    if constexpr (R1 != 0) {
      if constexpr (F::WAVE) sync16<N>();
      dft16<R1, true>(v, w1);
      exchange16<N, R1, R0>(v, ts, b1);
    }
    dft16<16, true>(v, w2);
    // Mirror: Z[N - k] of channel k = ts + r T is register 15 - r of thread T - ts (of thread 0: its own 16 - r).
    if constexpr (F::WAVE) sync16<N>();
#pragma unroll
    for (int i = 0; i < 8; ++i) b0[i * T + ts] = v[8 + i];
    sync16<N>();
    if (SPW == 1 || j < n_loc) {
#pragma unroll
      for (int r = 0; r < 8; ++r) {
        const float2 m = b0[(7 - r) * T + (ts ? T - ts : 0)];
        const float2 A = v[r], own = r ? v[16 - r] : v[0];
        const float2 B = ts ? m : own;
        // A + conj B = 2 X, A - conj B = 2i Y; 4 XX*, 4 YY*, 4 XY* (as the row pass)
        const float sx_ = A.x + B.x, sy_ = A.y - B.y;
        const float dx_ = A.x - B.x, dy_ = A.y + B.y;
        sum[0][r] += (double)(sx_ * sx_ + sy_ * sy_);
        sum[1][r] += (double)(dx_ * dx_ + dy_ * dy_);
        sum[2][r] += (double)(sx_ * dy_ - sy_ * dx_);
        sum[3][r] += (double)(sx_ * dx_ + sy_ * dy_);
      }
    }
    if constexpr (F::WAVE) sync16<N>();
  }
  // The slot in its layout, two products at a time through LDS (one pad per N1 channels), so that the stores of a
  // row are consecutive: the threads' channels alone lie N2 * 4 doubles apart.
  const int sh = 31 - __builtin_clz((unsigned)a.N1), half_len = N / 2 + (N / 2 >> sh);
  double* const d = reinterpret_cast<double*>(buf[sub][0]);
#pragma unroll
  for (int h = 0; h < 2; ++h) {
    if constexpr (F::WAVE) sync16<N>();
    else __syncthreads();
#pragma unroll
    for (int r = 0; r < 8; ++r) {
      const int k = ts + r * T;
      d[k + (k >> sh)] = sum[2 * h][r];
      d[half_len + k + (k >> sh)] = sum[2 * h + 1][r];
    }
    sync16<N>();
    if (n_loc) {
#pragma unroll
      for (int r = 0; r < 8; ++r) {
        const int e = ts + r * T, u = e / L, s = e & (L - 1);  // slot s of unit u
        const int half = s >= L / 2 ? 1 : 0, k2 = s - half * (L / 2);
        const int row = u == 0 ? half * U : (half ? a.N1 - u : u);
        const int k = row + (k2 << sh), o = (p * U + u) * 4 * L + s;
        slot[o + 2 * h * L] = d[k + (k >> sh)];
        slot[o + (2 * h + 1) * L] = d[half_len + k + (k >> sh)];
      }
    }
  }
}

template <int N, int BITS>
void fused_mode(int mode, const FusedArgs& a, const Launch& l) {
  constexpr int NT = fused_nt<N>(), SPW = 16 * NT / N;
  const dim3 grid((unsigned)((a.G + SPW - 1) / SPW), (unsigned)a.P), block(NT);
  if constexpr (BITS <= 8) {
    if (mode == 1) {
      hipExtLaunchKernelGGL((k_fused<N, BITS, 1>), grid, block, 0, l.stream, l.start, l.stop, 0, a);
      return;
    }
    if (mode == 2) {
      hipExtLaunchKernelGGL((k_fused<N, BITS, 2>), grid, block, 0, l.stream, l.start, l.stop, 0, a);
      return;
    }
  }
  hipExtLaunchKernelGGL((k_fused<N, BITS, 0>), grid, block, 0, l.stream, l.start, l.stop, 0, a);
}

template <int N>
hipError_t fused_bits(int bits, int mode, const FusedArgs& a, const Launch& l) {
  switch (bits) {
    case 2: fused_mode<N, 2>(mode, a, l); break;
    case 4: fused_mode<N, 4>(mode, a, l); break;
    case 8: fused_mode<N, 8>(mode, a, l); break;
    case 32: fused_mode<N, 32>(0, a, l); break;
    default: return hipErrorInvalidValue;
  }
  return hipGetLastError();
}

// stage 1: part[c][e] = sum of slots c*kReduceChunk .. in order; stage 2: out[e] = sum of part[c][e] in order
__global__ void __launch_bounds__(256) k_slot_chunks(const double* __restrict__ acc, int64_t elems, int slots,
                                                     int64_t slot_stride, double* __restrict__ part) {
  const int64_t e = (int64_t)blockIdx.x * 256 + threadIdx.x;
  const int c = (int)blockIdx.y;
  if (e >= elems) return;
  const int g1 = min(slots, (c + 1) * kReduceChunk);
  double s = 0.0;
#pragma unroll 8
  for (int g = c * kReduceChunk; g < g1; ++g) s += acc[(int64_t)g * slot_stride + e];  // loads issue 8 at a time
  part[(int64_t)c * elems + e] = s;
}

__global__ void __launch_bounds__(256) k_slot_total(const double* __restrict__ part, int64_t elems, int chunks,
                                                    double* __restrict__ out) {
  const int64_t e = (int64_t)blockIdx.x * 256 + threadIdx.x;
  if (e >= elems) return;
  double s = 0.0;
#pragma unroll 8
  for (int c = 0; c < chunks; ++c) s += part[(int64_t)c * elems + e];
  out[e] = s;
}

}  // namespace

hipError_t launch_slot_reduce(const double* acc, int64_t elems, int slots, int64_t slot_stride, double* part,
                              double* out, const Launch& l) {
  const int chunks = (int)slot_reduce_chunks(slots);
  const unsigned gx = (unsigned)((elems + 255) / 256);
  hipExtLaunchKernelGGL(k_slot_chunks, dim3(gx, (unsigned)chunks), dim3(256), 0, l.stream, l.start,
                        out ? nullptr : l.stop, 0, acc, elems, slots, slot_stride, part);
  if (out)
    hipExtLaunchKernelGGL(k_slot_total, dim3(gx), dim3(256), 0, l.stream, nullptr, l.stop, 0, part, elems, chunks, out);
  return hipGetLastError();
}

hipError_t launch_fused(int N, int bits, int mode, const FusedArgs& a, const Launch& l) {
  // the word loaders need words that are aligned in the buffer (frames start at multiples of 32 samples or more)
  const unsigned word = mode ? (unsigned)(a.S * bits / 8) : 1u;
  if (word > 1 && reinterpret_cast<uintptr_t>(a.in) % word) mode = 0;
  switch (N) {
    case 1 << 8: return fused_bits<1 << 8>(bits, mode, a, l);
    case 1 << 9: return fused_bits<1 << 9>(bits, mode, a, l);
    case 1 << 10: return fused_bits<1 << 10>(bits, mode, a, l);
    case 1 << 11: return fused_bits<1 << 11>(bits, mode, a, l);
    case 1 << 12: return fused_bits<1 << 12>(bits, mode, a, l);
    default: return hipErrorInvalidValue;
  }
}

}  // namespace ps
