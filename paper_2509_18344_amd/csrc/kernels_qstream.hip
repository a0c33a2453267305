// The substitute-layer linear y = x * dequant(q, s, z)^T (SubSpec Sec. 4.1) for draft
// batches of up to 16 tree tokens (k_qstream): the weight stream is all the work there,
// so a workgroup takes NT tiles of 16 columns over the whole of K and its KS wavefronts
// take the 128-k blocks in turn (wavefront w blocks w, w + KS, ...).  Nothing is shared
// until the end: no activations staged in LDS, no barrier in the loop and no partial sums
// in memory, whose completion (stores acknowledged, counter, reads by the last workgroup)
// is three trips to the coherent level in a row.  The wavefronts' sums meet once in LDS.
//
// One block: 16x16x32 bf16 MFMAs, A = x fragments loaded from memory straight into the
// operand layout (x is small and stays in the L2; rows past M are outside the buffer
// resource and read zeros without traffic; up to 4 or 8 rows one or two loads hold all four
// steps and DPP moves spread them: 7168x5120 3-bit M = 1 7.0 us with four loads, 5.7 with one), B = unpacked codes 128 + q, and one more MFMA
// per step with B = 1 for the group's sum of x, which lands in the accumulator's layout:
//     tot += s * ( sum x (128+q) - (128+z) * sum x ).
// The weights, scales and activations of PF blocks are in flight per wavefront.
//
// Neighbouring column groups share cache lines of the scales (a line holds 64 columns),
// so the grid is dealt to the eight XCDs in contiguous runs of column groups.
//
// What bounds it: the latency of the launch, of one or two rounds of loads per wavefront
// and of the meeting in LDS (4608x3584 4-bit, 8.8 MB: 7.7 us split across workgroups with
// its completion, 4.6 here, against some 3.2 for an empty launch and the bytes), and with
// more rows the address units, which take 16 cycles per load of any size: four of x and
// two to four of scales stand beside each kilobyte of codes.
#include "kernels_qstream.h"
#include "qlinear_device.h"

namespace subspec {

namespace {

constexpr int kXcds = 8;

template <int BITS, int GROUP, int NT, int KS, int PF, int AL>
struct StreamBody {
  static constexpr int GPB = kTileK / GROUP;  // groups per block
  static constexpr int SPG = 4 / GPB;         // 32-k steps per group
  struct Ring {
    Slice<BITS> w[NT];
    uint16_t s[GPB][NT], z[GPB][NT];
    u32x4_t a[AL];
  };

  static __device__ __forceinline__ void load(Ring& r, const QBuffers& bu, int N, const uint32_t (&wofs)[NT],
                                              const uint32_t (&szofs)[NT], uint32_t xofs, int kb) {
#pragma unroll
    for (int t = 0; t < NT; ++t) r.w[t] = load_slice<BITS>(bu.w, wofs[t] + static_cast<uint32_t>(kb) * (256 * BITS));
#pragma unroll
    for (int i = 0; i < AL; ++i)
      r.a[i] = __builtin_bit_cast(u32x4_t, __builtin_amdgcn_raw_buffer_load_b128(bu.x, xofs + 256 / AL * i, kb * (kTileK * 2), 0));
#pragma unroll
    for (int gi = 0; gi < GPB; ++gi) {
      const uint32_t soff = static_cast<uint32_t>(kb * GPB + gi) * N * 2;
#pragma unroll
      for (int t = 0; t < NT; ++t) {
        r.s[gi][t] = __builtin_amdgcn_raw_buffer_load_b16(bu.s, szofs[t], soff, 0);
        r.z[gi][t] = __builtin_amdgcn_raw_buffer_load_b16(bu.z, szofs[t], soff, 0);
      }
    }
  }

  // A fragment of 32-k step J.  One load holds it for 4 / AL steps: lane 16 q + 4 AL i + row
  // has the row's piece q of the load's step i (at most 4 AL rows), so the lanes of a row of 16
  // move down by 4 AL i.  The fragment's rows past 4 AL then hold other steps' pieces: their
  // outputs are never stored.
  template <int J>
  static __device__ __forceinline__ bf16x8_t fragment(const Ring& r) {
    constexpr int PER = 4 / AL, I = J % PER;  // steps per load
    u32x4_t v = r.a[J / PER];
    if constexpr (I > 0) {
#pragma unroll
      for (int e = 0; e < 4; ++e) {
        const int w = static_cast<int>(v[e]);
        v[e] = static_cast<uint32_t>(__builtin_amdgcn_update_dpp(0, w, 0x100 | (4 * AL * I), 0xF, 0xF, true));  // row_shl
      }
    }
    return __builtin_bit_cast(bf16x8_t, v);
  }

  static __device__ __forceinline__ void compute(const Ring& r, f32x4_t (&tot)[NT]) {
    const bf16x8_t ones = __builtin_bit_cast(bf16x8_t, make_uint4(0x3F803F80u, 0x3F803F80u, 0x3F803F80u, 0x3F803F80u));
    const f32x4_t zero = f32x4_t{0.f, 0.f, 0.f, 0.f};
    static_for<GPB>([&](auto gc) __attribute__((always_inline)) {
      constexpr int gi = decltype(gc)::value;
      f32x4_t acc[NT], accx;
      static_for<SPG>([&](auto sc) __attribute__((always_inline)) {
        constexpr int js = decltype(sc)::value, j = gi * SPG + js;
        const bf16x8_t A = fragment<j>(r);
        accx = __builtin_amdgcn_mfma_f32_16x16x32_bf16(A, ones, js == 0 ? zero : accx, 0, 0, 0);
#pragma unroll
        for (int t = 0; t < NT; ++t)
          acc[t] = __builtin_amdgcn_mfma_f32_16x16x32_bf16(A, b_operand<BITS, j>(r.w[t]), js == 0 ? zero : acc[t], 0, 0, 0);
      });
#pragma unroll
      for (int t = 0; t < NT; ++t) {
        const float s = half_bits_to_float(r.s[gi][t]);
        const float nz = -(kCodeBias + half_bits_to_float(r.z[gi][t]));
#pragma unroll
        for (int e = 0; e < 4; ++e)
          tot[t][e] = __builtin_fmaf(s, __builtin_fmaf(nz, accx[e], acc[t][e]), tot[t][e]);
      }
    });
  }
};

template <int BITS, int GROUP, int NT, int KS, int PF, int AL>
__global__ __launch_bounds__(KS * kWave) void k_qstream(QArgs a) {
  using Body = StreamBody<BITS, GROUP, NT, KS, PF, AL>;
  __shared__ float red[KS][NT * 4][kWave];
  const int lane = threadIdx.x % kWave;
  const int wave = __builtin_amdgcn_readfirstlane(static_cast<int>(threadIdx.x / kWave));
  const int groups = (a.n_tiles + NT - 1) / NT;
  // XCD x (workgroups x, x + 8, ...) takes groups [x * per, x * per + per).
  const int per = (groups + kXcds - 1) / kXcds;
  const int ng = static_cast<int>(blockIdx.x % kXcds) * per + static_cast<int>(blockIdx.x / kXcds);
  if (ng >= groups || static_cast<int>(blockIdx.x / kXcds) >= per) return;  // the whole workgroup
  const QBuffers bu(a, BITS, GROUP);

  uint32_t wofs[NT], szofs[NT];
#pragma unroll
  for (int t = 0; t < NT; ++t) {
    const int nt = min(ng * NT + t, a.n_tiles - 1);  // tiles past N repeat the last one, never stored
    wofs[t] = static_cast<uint32_t>(nt) * a.KB * (256 * BITS) + lane * (4 * BITS);
    szofs[t] = static_cast<uint32_t>(nt * kTileN + (lane & 15)) * 2;
  }
  // Row lane % (4 AL), piece lane / 16 of the step lane / (4 AL) % (4 / AL) of each load.
  const uint32_t xofs = (static_cast<uint32_t>(lane % (4 * AL)) * a.K + lane / (4 * AL) % (4 / AL) * 32 + 8 * (lane >> 4)) * 2;
  // This wavefront's blocks: first + i * KS, i < n.  Loads past the last repeat it (and a
  // wavefront without blocks loads one it never uses), so that every load is unconditional.
  const int n = wave < a.KB ? (a.KB - wave + KS - 1) / KS : 0;
  const int first = min(wave, a.KB - 1), lasti = max(n - 1, 0);
  f32x4_t tot[NT];
#pragma unroll
  for (int t = 0; t < NT; ++t) tot[t] = f32x4_t{0.f, 0.f, 0.f, 0.f};

  typename Body::Ring ring[PF];
  static_for<PF>([&](auto u) __attribute__((always_inline)) {
    Body::load(ring[u.value], bu, a.N, wofs, szofs, xofs, first + min(static_cast<int>(u.value), lasti) * KS);
  });
  int c = 0;
  for (; c + PF < n; c += PF)
    static_for<PF>([&](auto u) __attribute__((always_inline)) {
      Body::compute(ring[u.value], tot);
      Body::load(ring[u.value], bu, a.N, wofs, szofs, xofs, first + min(c + static_cast<int>(u.value) + PF, lasti) * KS);
    });
  static_for<PF>([&](auto u) __attribute__((always_inline)) {
    if (c + static_cast<int>(u.value) < n) Body::compute(ring[u.value], tot);
  });

  // The wavefronts' sums, added in wavefront order.  D layout of the 16x16 MFMA: lane
  // holds column lane % 16, rows 4 (lane / 16) + e.
#pragma unroll
  for (int t = 0; t < NT; ++t)
#pragma unroll
    for (int e = 0; e < 4; ++e) red[wave][4 * t + e][lane] = tot[t][e];
  __syncthreads();
  for (int i = threadIdx.x; i < NT * 4 * kWave; i += KS * kWave) {
    const int v = i / kWave, ln = i % kWave;
    const int m = 4 * (ln >> 4) + (v & 3), nt = ng * NT + v / 4;
    if (m >= a.M || nt >= a.n_tiles) continue;
    float sum = red[0][v][ln];
#pragma unroll
    for (int w = 1; w < KS; ++w) sum += red[w][v][ln];
    a.y[static_cast<size_t>(m) * a.N + nt * kTileN + (ln & 15)] = float_to_bf16_bits(sum);
  }
}

typedef void (*StreamKernel)(QArgs);
struct StreamVariant {
  int bits, group, nt, ks, al, ring;
  StreamKernel fn;
};
// P1, P: blocks in flight with one load of x per block and with more (sixteen wavefronts
// per CU leave 128 registers each).
#define SUBSPEC_STREAM(B, G, T, W, P1, P)                                                            \
  {B, G, T, W, 1, P1, k_qstream<B, G, T, W, P1, 1>}, {B, G, T, W, 2, P, k_qstream<B, G, T, W, P, 2>}, \
      {B, G, T, W, 4, P, k_qstream<B, G, T, W, P, 4>}
#define SUBSPEC_STREAM_SET(B, G)                                                \
  SUBSPEC_STREAM(B, G, 1, 4, 3, 3), SUBSPEC_STREAM(B, G, 1, 16, 4, 3),          \
      SUBSPEC_STREAM(B, G, 2, 8, 3, 3), SUBSPEC_STREAM(B, G, 2, 16, 2, 2),
const StreamVariant kVariants[] = {SUBSPEC_STREAM_SET(4, 128) SUBSPEC_STREAM_SET(4, 64) SUBSPEC_STREAM_SET(3, 128)
                                       SUBSPEC_STREAM_SET(3, 64) SUBSPEC_STREAM_SET(2, 128) SUBSPEC_STREAM_SET(2, 64)};

const StreamVariant* find_stream(int nt, int ks, int bits, int group, int M) {
  const int al = M <= 4 ? 1 : M <= 8 ? 2 : 4;  // loads of x per block
  for (const StreamVariant& v : kVariants)
    if (v.nt == nt && v.ks == ks && v.al == al && v.bits == bits && v.group == group) return &v;
  return nullptr;
}

}  // namespace

int qstream_ring(int nt, int ks, int bits, int group, int M) {
  const StreamVariant* v = find_stream(nt, ks, bits, group, M);
  return v ? v->ring : 0;
}

int qstream_grid(int groups) { return (groups + kXcds - 1) / kXcds * kXcds; }

hipError_t launch_qstream(int nt, int ks, int bits, int group, const QArgs& a, hipStream_t st) {
  const StreamVariant* v = find_stream(nt, ks, bits, group, a.M);
  if (!v) return hipErrorInvalidDeviceFunction;
  hipLaunchKernelGGL(v->fn, dim3(qstream_grid((a.n_tiles + nt - 1) / nt)), dim3(ks * kWave), 0, st, a);
  return hipGetLastError();
}

}  // namespace subspec
