// Weight preparation kernels: min/max quantizer, the quantizer with an HQQ-style
// optimised zero-point, packer into the tile layout and the materialising
// dequantizer (include/subspec.h documents each operation).
#include "device_common.h"
#include "kernels.h"
#include "kernels_hqq.h"

namespace subspec {

// float64 -> IEEE binary16 bits, round to nearest, ties to even, written from the
// format definition: 1 sign bit, 5 exponent bits (bias 15), 10 fraction bits,
// subnormals below 2^-14, overflow to infinity.
__device__ __forceinline__ uint16_t f64_to_f16_bits(double d) {
  const uint64_t u = __builtin_bit_cast(uint64_t, d);
  const uint16_t sign = static_cast<uint16_t>((u >> 48) & 0x8000u);
  const int ex = static_cast<int>((u >> 52) & 0x7FF);
  const uint64_t frac = u & ((1ull << 52) - 1);
  if (ex == 0x7FF) return sign | 0x7C00u | (frac ? 0x200u : 0u);  // inf / NaN
  if (ex == 0) return sign;                   // float64 zero or subnormal: |d| < 2^-1022
  const int e = ex - 1023;                    // d = 1.frac * 2^e
  if (e > 15) return sign | 0x7C00u;          // >= 2^16: overflow
  if (e < -25) return sign;                   // < 2^-25: rounds to zero
  const uint64_t sig = (1ull << 52) | frac;   // 53-bit significand
  // Keep 11 bits for normal results; fewer for subnormal ones (quantum 2^-24).
  const int shift = (e >= -14) ? 42 : 42 + (-14 - e);
  uint64_t m = sig >> shift;
  const uint64_t rem = sig & ((1ull << shift) - 1);
  const uint64_t half = 1ull << (shift - 1);
  if (rem > half || (rem == half && (m & 1))) ++m;
  if (e >= -14) {
    // m in [2^10, 2^11]; a carry to 2^11 bumps the exponent (and may reach inf).
    return sign | static_cast<uint16_t>(((e + 15 - 1) << 10) + m);
  }
  return sign | static_cast<uint16_t>(m);     // subnormal (m == 2^10 is the min normal)
}

__device__ __forceinline__ double f16_bits_to_f64(uint16_t h) {
  return static_cast<double>(__builtin_bit_cast(_Float16, h));
}

// One wavefront per (column n, group g).  Lane l holds GROUP/64 consecutive values.
template <int GROUP>
__global__ __launch_bounds__(256) void k_quantize(const float* __restrict__ w, int bits,
                                                  int N, int K, uint8_t* __restrict__ codes,
                                                  uint16_t* __restrict__ sc,
                                                  uint16_t* __restrict__ zr) {
  constexpr int PER = GROUP / kWave;
  const int gpr = K / GROUP;
  const long long gid = static_cast<long long>(blockIdx.x) * 4 + threadIdx.x / kWave;
  if (gid >= static_cast<long long>(N) * gpr) return;  // whole wavefronts exit together
  const int lane = threadIdx.x % kWave;
  const long long n = gid / gpr;
  const int g = static_cast<int>(gid % gpr);
  const float* src = w + n * K + static_cast<long long>(g) * GROUP + lane * PER;
  float v[PER];
#pragma unroll
  for (int i = 0; i < PER; ++i) v[i] = src[i];
  float mn = v[0], mx = v[0];
#pragma unroll
  for (int i = 1; i < PER; ++i) { mn = fminf(mn, v[i]); mx = fmaxf(mx, v[i]); }
#pragma unroll
  for (int off = 32; off >= 1; off >>= 1) {
    mn = fminf(mn, __shfl_xor(mn, off));
    mx = fmaxf(mx, __shfl_xor(mx, off));
  }
  const double wmin = mn, wmax = mx;
  const double qmax = static_cast<double>((1 << bits) - 1);
  uint16_t s16 = f64_to_f16_bits((wmax - wmin) / qmax);
  double s = f16_bits_to_f64(s16);
  const bool degenerate = (wmax == wmin) || (s == 0.0);
  uint16_t z16;
  if (degenerate) {
    s16 = 0x3C00u;
    s = 1.0;
    z16 = f64_to_f16_bits(-wmin);
  } else {
    z16 = f64_to_f16_bits(-wmin / s);
  }
  const double z = f16_bits_to_f64(z16);
  uint8_t* dst = codes + n * K + static_cast<long long>(g) * GROUP + lane * PER;
#pragma unroll
  for (int i = 0; i < PER; ++i) {
    double t = static_cast<double>(v[i]) / s + z;
    t = __builtin_rint(t);
    t = t < 0.0 ? 0.0 : (t > qmax ? qmax : t);
    dst[i] = degenerate ? 0 : static_cast<uint8_t>(t);
  }
  if (lane == 0) {
    sc[static_cast<long long>(g) * N + n] = s16;
    zr[static_cast<long long>(g) * N + n] = z16;
  }
}

// HQQ-style zero-point (SubSpec Sec. 4.1 and 5.1 quantize the substitutes with HQQ;
// the rounds follow the cited half-quadratic quantization work).  The scale is the
// min/max scale; starting from the min/max zero, each round quantizes with the
// current zero, shrinks the residual x = w - s (q - z) with the generalised soft
// threshold sign(x) max(|x| - |x|^(p-1) / beta, 0) and refits the zero as the mean of
// q - (w - e) / s; the group's sum of |w - s (q - z)| decides: the best zero is kept
// and a round without improvement ends the search; beta grows by kappa per round.
// The best zero, rounded to fp16, replaces the min/max zero only if it is still
// better in fp16.  Everything in float64 with sums in index order, one thread per
// (column n, group g), so that the rounding decisions are reproducible.
constexpr double kHqqP = 0.7;
constexpr double kHqqBeta = 10.0;
constexpr double kHqqKappa = 1.01;
constexpr int kHqqIters = 20;

// What bounds it, and the layout.  The rounds are float64 arithmetic; a float64 division
// costs about as much as the rest of an element's step and the power function several
// times that, so both leave the rounds (7B down, 3584 x 18944, 4-bit groups of 64:
// 7000 us with them):
//  - w / s does not change from round to round: the quotients are computed once.
//  - the residual x of an unclamped weight is at most s / 2, where the soft threshold is
//    zero: |x| - |x|^(p-1) / beta > 0 needs |x|^(2-p) > 1 / beta.  For |x| <= kHqqNoShrink
//    it cannot hold in any round (the largest beta of the rounds is 12.2, and
//    0.125^(p-1) / 12.2 = 0.153 > 0.125, a margin far beyond rounding): e is zero and
//    the refitted term is q - w / s.  A group that meets a larger residual starts over with
//    the plain rounds (hqq_group).  (A NaN among the weights leaves no error sum below the
//    first one in either form, so the min/max zero stays.)
//  - the error sum of a new zero and the next refit need the same codes: one pass
//    computes both (the refit of the last pass is not used).
// Every value that decides anything comes from the same operations in the same order as
// in the plain rounds, so the results are bit for bit theirs.  One thread works on one
// group, since its sums run in index order, with the weights and quotients in registers
// (in LDS they would leave less than one wavefront per SIMD).
constexpr double kHqqNoShrink = 0.125;

__device__ __forceinline__ double hqq_code(double quot, double z, double qmax) {
  const double c = __builtin_rint(quot + z);
  return c < 0.0 ? 0.0 : (c > qmax ? qmax : c);
}

__device__ __forceinline__ uint32_t hqq_word(const double* quot, double z, double qmax) {
  uint32_t b = 0;
#pragma unroll
  for (int k = 0; k < 4; ++k) b |= static_cast<uint32_t>(hqq_code(quot[k], z, qmax)) << (8 * k);
  return b;
}

// The plain rounds for one group from its weights in memory: returns the zero's fp16
// bits and stores the codes.  W elements at a time: one or two wavefronts per SIMD leave
// a float64 power's chain of operations exposed otherwise.  W residuals within
// kHqqNoShrink in every lane need no power.  W is four for groups of 64, where eight would
// take the registers of the second wavefront (3584 x 3584, every group beyond the bound:
// 2680 us against 3050; one element at a time 3050, all rounds in this form with the weights
// in LDS 2610; 3584 x 18944 10800 us, in LDS 11100), and eight for groups of 128
// (3584 x 3584 3190 us against 3310; one element at a time 4030, in LDS 4280).
template <int W>
__device__ __attribute__((noinline)) uint16_t hqq_group(const float* src, uint8_t* dst, int group, double s,
                                                        uint16_t z16, double qmax) {
  // W elements' weights, quotients, codes and residuals under zero z
  struct Part {
    double x[W], quot[W], q[W], r[W];
    __device__ __forceinline__ Part(const float* p, double s, double z, double qmax) {
#pragma unroll
      for (int k = 0; k < W; k += 4) {
        const float4 f = *reinterpret_cast<const float4*>(p + k);
        x[k] = f.x, x[k + 1] = f.y, x[k + 2] = f.z, x[k + 3] = f.w;
      }
#pragma unroll
      for (int k = 0; k < W; ++k) {
        quot[k] = x[k] / s;
        q[k] = hqq_code(quot[k], z, qmax);
        r[k] = x[k] - (q[k] - z) * s;
      }
    }
  };
  auto l1 = [&](double z) {
    double tot = 0.0;
    for (int i = 0; i < group; i += W) {
      const Part v(src + i, s, z, qmax);
#pragma unroll
      for (int k = 0; k < W; ++k) tot += fabs(v.r[k]);
    }
    return tot;
  };
  const double z0 = f16_bits_to_f64(z16);
  double z = z0, best_z = z0, best = 0.0, e0 = 0.0, beta = kHqqBeta;
  for (int it = 0; it < kHqqIters; ++it) {
    double acc = 0.0, tot = 0.0;  // the refit sum, and the error sum of the zero it starts from
    for (int i = 0; i < group; i += W) {
      const Part v(src + i, s, z, qmax);
      double t[W];
      bool within = true;
#pragma unroll
      for (int k = 0; k < W; ++k) {
        t[k] = v.quot[k];
        within = within && fabs(v.r[k]) <= kHqqNoShrink;
      }
      if (__ballot(!within)) {
#pragma unroll
        for (int k = 0; k < W; ++k) {
          const double a = fabs(v.r[k]);
          const double e = v.r[k] == 0.0 ? 0.0 : copysign(fmax(a - pow(a, kHqqP - 1.0) / beta, 0.0), v.r[k]);
          t[k] = (v.x[k] - e) / s;
        }
      }
#pragma unroll
      for (int k = 0; k < W; ++k) {
        acc += v.q[k] - t[k];
        tot += fabs(v.r[k]);
      }
    }
    if (it == 0) e0 = best = tot;
    const double z_new = acc / group;
    const double err = l1(z_new);
    if (!(err < best)) break;
    best = err;
    best_z = z_new;
    z = z_new;
    beta = beta * kHqqKappa;
  }
  const uint16_t zb = f64_to_f16_bits(best_z);
  if (l1(f16_bits_to_f64(zb)) < e0) z16 = zb;
  const double zf = f16_bits_to_f64(z16);
  for (int i = 0; i < group; i += W) {
    const Part v(src + i, s, zf, qmax);
#pragma unroll
    for (int k = 0; k < W; k += 4) *reinterpret_cast<uint32_t*>(dst + i + k) = hqq_word(v.quot + k, zf, qmax);
  }
  return z16;
}

template <int GROUP>
__global__ __launch_bounds__(kWave) __attribute__((amdgpu_waves_per_eu(GROUP == 64 ? 2 : 1))) void k_quantize_hqq(const float* __restrict__ w, int bits, int N, int K,
                                                       uint8_t* __restrict__ codes, uint16_t* __restrict__ sc,
                                                       uint16_t* __restrict__ zr) {
  const int gpr = K / GROUP;
  const long long gid = static_cast<long long>(blockIdx.x) * kWave + threadIdx.x;  // g * N + n
  if (gid >= static_cast<long long>(N) * gpr) return;
  const long long n = gid % N;
  const int g = static_cast<int>(gid / N);
  const float* src = w + n * K + static_cast<long long>(g) * GROUP;
  float wv[GROUP];
  float mn = INFINITY, mx = -INFINITY;
#pragma unroll
  for (int i = 0; i < GROUP; i += 4) {
    const float4 q4 = *reinterpret_cast<const float4*>(src + i);
    wv[i] = q4.x;
    wv[i + 1] = q4.y;
    wv[i + 2] = q4.z;
    wv[i + 3] = q4.w;
    mn = fminf(fminf(mn, q4.x), fminf(fminf(q4.y, q4.z), q4.w));
    mx = fmaxf(fmaxf(mx, q4.x), fmaxf(fmaxf(q4.y, q4.z), q4.w));
  }
  const double wmin = mn, wmax = mx;
  const double qmax = static_cast<double>((1 << bits) - 1);
  uint16_t s16 = f64_to_f16_bits((wmax - wmin) / qmax);
  double s = f16_bits_to_f64(s16);
  const bool degenerate = (wmax == wmin) || (s == 0.0);
  uint16_t z16;
  if (degenerate) {
    s16 = 0x3C00u;
    s = 1.0;
    z16 = f64_to_f16_bits(-wmin);
  } else {
    z16 = f64_to_f16_bits(-wmin / s);
  }
  // Residuals of unclamped weights spread over half a scale: with a scale well above twice
  // the bound one of them passes it all but surely, and the group starts with the plain rounds.
  bool large = !degenerate && s > 2.4 * kHqqNoShrink;
  double quot[GROUP];
  if (!large) {
#pragma unroll
    for (int i = 0; i < GROUP; ++i) {
      quot[i] = static_cast<double>(wv[i]) / s;
      asm volatile("" : "+v"(quot[i]));
    }
  }
  // The error sum of zero z, and the refit sum of the round that starts from it.
  auto pass = [&](double z, double& refit) __attribute__((always_inline)) {
    double err = 0.0, acc = 0.0, amax = 0.0;
#pragma unroll
    for (int i = 0; i < GROUP; ++i) {
      const double q = hqq_code(quot[i], z, qmax);
      double x;  // converted in every pass: kept across passes, it would take two registers more
      asm volatile("v_cvt_f64_f32 %0, %1" : "=v"(x) : "v"(wv[i]));
      const double a = fabs(x - (q - z) * s);
      err += a;
      acc += q - quot[i];
      amax = fmax(amax, a);
      // four elements at a time: with all 64 in flight the values spill
      if (i % 4 == 3) asm volatile("" : "+v"(err), "+v"(acc), "+v"(amax));
    }
    refit = acc;
    large = !(amax <= kHqqNoShrink);
    return err;
  };
  if (!degenerate && !large) {
    const double z0 = f16_bits_to_f64(z16);
    // Pass 0 is the min/max zero, pass p > 0 the zero of round p - 1; the pass after the
    // search ended is the best zero in fp16.  One copy of the unrolled pass serves all.
    double z = z0, best_z = z0, best = 0.0, e0 = 0.0;
    for (int p = 0;; ++p) {
      double refit;
      const double err = pass(z, refit);
      if (large) break;
      if (p > kHqqIters + 1) {  // z is the best zero rounded to fp16
        if (err < e0) z16 = f64_to_f16_bits(z);
        break;
      }
      bool more = p < kHqqIters;
      if (p == 0) {
        e0 = best = err;
      } else if (err < best) {
        best = err;
        best_z = z;
      } else {
        more = false;
      }
      if (more) {
        z = refit / GROUP;
      } else {
        z = f16_bits_to_f64(f64_to_f16_bits(best_z));
        p = kHqqIters + 1;  // the last pass follows
      }
    }
  }
  uint8_t* dst = codes + n * K + static_cast<long long>(g) * GROUP;
  if (large) {
    z16 = hqq_group<GROUP == 64 ? 4 : 8>(src, dst, GROUP, s, z16, qmax);
  } else {
    const double zf = f16_bits_to_f64(z16);
#pragma unroll
    for (int i = 0; i < GROUP; i += 16) {
      uint32_t word[4];
#pragma unroll
      for (int j = 0; j < 4; ++j) word[j] = degenerate ? 0u : hqq_word(quot + i + 4 * j, zf, qmax);
      __builtin_amdgcn_sched_barrier(0);
      *reinterpret_cast<uint4*>(dst + i) = make_uint4(word[0], word[1], word[2], word[3]);
    }
  }
  sc[static_cast<long long>(g) * N + n] = s16;
  zr[static_cast<long long>(g) * N + n] = z16;
}

// Packed words of one slice from its 32 codes c[e + 8*j] (k order of the slice).
template <int BITS>
__device__ __forceinline__ void pack_slice_words(const uint32_t c[32], uint32_t* out) {
  constexpr uint32_t mask = (1u << BITS) - 1;
  for (int w = 0; w < BITS; ++w) out[w] = 0;
#pragma unroll
  for (int p = 0; p < 16; ++p) {
    const int j = p / 4, i = p % 4;
    const uint32_t ev = c[8 * j + 2 * i] & mask, od = c[8 * j + 2 * i + 1] & mask;
    if constexpr (BITS == 4) {
      out[p / 4] |= (ev << (4 * (p % 4))) | (od << (16 + 4 * (p % 4)));
    } else if constexpr (BITS == 2) {
      out[p / 8] |= (ev << (2 * (p % 8))) | (od << (16 + 2 * (p % 8)));
    } else {
      if (p < 15) {
        out[p / 5] |= (ev << (3 * (p % 5))) | (od << (16 + 3 * (p % 5)));
      } else {
#pragma unroll
        for (int b = 0; b < 3; ++b)
          out[b] |= (((ev >> b) & 1u) << 15) | (((od >> b) & 1u) << 31);
      }
    }
  }
}

// One thread per (tile, slice).
template <int BITS>
__global__ __launch_bounds__(256) void k_qpack(const uint8_t* __restrict__ codes, int N, int K,
                                               uint8_t* __restrict__ qw) {
  const int KB = K / kTileK;
  const long long tiles = static_cast<long long>(N / kTileN) * KB;
  const long long gidx = static_cast<long long>(blockIdx.x) * blockDim.x + threadIdx.x;
  if (gidx >= tiles * kWave) return;
  const long long tile = gidx / kWave;
  const int L = static_cast<int>(gidx % kWave);
  const long long nt = tile / KB;
  const int kb = static_cast<int>(tile % KB);
  const long long n = nt * kTileN + L % 16;
  const uint8_t* row = codes + n * K + kb * kTileK + 8 * (L / 16);
  uint32_t c[32];
#pragma unroll
  for (int j = 0; j < 4; ++j) {
    const uint2 v = *reinterpret_cast<const uint2*>(row + 32 * j);
#pragma unroll
    for (int e = 0; e < 4; ++e) {
      c[8 * j + e] = (v.x >> (8 * e)) & 0xFFu;
      c[8 * j + 4 + e] = (v.y >> (8 * e)) & 0xFFu;
    }
  }
  uint32_t words[BITS];
  pack_slice_words<BITS>(c, words);
  uint32_t* dst = reinterpret_cast<uint32_t*>(qw + (tile * kWave + L) * (4 * BITS));
#pragma unroll
  for (int w = 0; w < BITS; ++w) dst[w] = words[w];
}

// One thread per (tile, slice): unpack with the qlinear kernels' code, then dequant.
template <int BITS>
__global__ __launch_bounds__(256) void k_qdequant(const uint8_t* __restrict__ qw,
                                                  const uint16_t* __restrict__ sc,
                                                  const uint16_t* __restrict__ zr, int group,
                                                  int N, int K, float* __restrict__ wf,
                                                  uint16_t* __restrict__ wb) {
  const int KB = K / kTileK;
  const long long tiles = static_cast<long long>(N / kTileN) * KB;
  const long long gidx = static_cast<long long>(blockIdx.x) * blockDim.x + threadIdx.x;
  if (gidx >= tiles * kWave) return;
  const long long tile = gidx / kWave;
  const int L = static_cast<int>(gidx % kWave);
  const long long nt = tile / KB;
  const int kb = static_cast<int>(tile % KB);
  const long long n = nt * kTileN + L % 16;
  const Slice<BITS> s = load_slice<BITS>(qw + (tile * kWave + L) * (4 * BITS));
  uint32_t pr[16];
  unpack_pairs<BITS>(s, pr);
#pragma unroll
  for (int p = 0; p < 16; ++p) {
    const int k0 = kb * kTileK + 32 * (p / 4) + 8 * (L / 16) + 2 * (p % 4);
#pragma unroll
    for (int h = 0; h < 2; ++h) {
      const int k = k0 + h;
      const float q = static_cast<float>((pr[p] >> (16 * h)) & 0xFFu);
      const long long gi = static_cast<long long>(k / group) * N + n;
      const float sv = half_bits_to_float(sc[gi]);
      const float zv = half_bits_to_float(zr[gi]);
      const float b = -(sv * zv);  // exact: product of two fp16 values
      const float v = __builtin_fmaf(q, sv, b);
      if (wf) wf[n * K + k] = v;
      if (wb) wb[n * K + k] = float_to_bf16_bits(v);
    }
  }
}

hipError_t launch_quantize(const float* w, int bits, int group, int N, int K, uint8_t* codes,
                           uint16_t* sc, uint16_t* zr, hipStream_t st) {
  const long long groups = static_cast<long long>(N) * (K / group);
  const long long blocks = (groups + 3) / 4;
  if (group == 64)
    hipLaunchKernelGGL(k_quantize<64>, dim3(static_cast<unsigned>(blocks)), dim3(256), 0, st, w,
                       bits, N, K, codes, sc, zr);
  else
    hipLaunchKernelGGL(k_quantize<128>, dim3(static_cast<unsigned>(blocks)), dim3(256), 0, st, w,
                       bits, N, K, codes, sc, zr);
  return hipGetLastError();
}

hipError_t launch_quantize_hqq(const float* w, int bits, int group, int N, int K, uint8_t* codes,
                               uint16_t* sc, uint16_t* zr, hipStream_t st) {
  const long long groups = static_cast<long long>(N) * (K / group);
  const dim3 grid(static_cast<unsigned>((groups + kWave - 1) / kWave)), block(kWave);
  if (group == 64)
    hipLaunchKernelGGL(k_quantize_hqq<64>, grid, block, 0, st, w, bits, N, K, codes, sc, zr);
  else
    hipLaunchKernelGGL(k_quantize_hqq<128>, grid, block, 0, st, w, bits, N, K, codes, sc, zr);
  return hipGetLastError();
}

hipError_t launch_qpack(const uint8_t* codes, int bits, int N, int K, void* qw, hipStream_t st) {
  const long long threads = static_cast<long long>(N / kTileN) * (K / kTileK) * kWave;
  const dim3 grid(static_cast<unsigned>((threads + 255) / 256));
  uint8_t* out = static_cast<uint8_t*>(qw);
  switch (bits) {
    case 4: hipLaunchKernelGGL(k_qpack<4>, grid, dim3(256), 0, st, codes, N, K, out); break;
    case 3: hipLaunchKernelGGL(k_qpack<3>, grid, dim3(256), 0, st, codes, N, K, out); break;
    default: hipLaunchKernelGGL(k_qpack<2>, grid, dim3(256), 0, st, codes, N, K, out); break;
  }
  return hipGetLastError();
}

hipError_t launch_qdequant(const void* qw, const void* sc, const void* zr, int bits, int group,
                           int N, int K, float* wf, uint16_t* wb, hipStream_t st) {
  const long long threads = static_cast<long long>(N / kTileN) * (K / kTileK) * kWave;
  const dim3 grid(static_cast<unsigned>((threads + 255) / 256));
  const uint8_t* q = static_cast<const uint8_t*>(qw);
  const uint16_t* s = static_cast<const uint16_t*>(sc);
  const uint16_t* z = static_cast<const uint16_t*>(zr);
  switch (bits) {
    case 4: hipLaunchKernelGGL(k_qdequant<4>, grid, dim3(256), 0, st, q, s, z, group, N, K, wf, wb); break;
    case 3: hipLaunchKernelGGL(k_qdequant<3>, grid, dim3(256), 0, st, q, s, z, group, N, K, wf, wb); break;
    default: hipLaunchKernelGGL(k_qdequant<2>, grid, dim3(256), 0, st, q, s, z, group, N, K, wf, wb); break;
  }
  return hipGetLastError();
}

}  // namespace subspec
