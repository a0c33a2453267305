// Tree attention of the draft model over the shared KV cache (SubSpec Sec. 4.1,
// "Shared KV-Cache"; tree masks as in Sec. 2 and Sec. 4.2).
//
// One draft pass of one decoder layer: M new tree tokens, each with Hq query heads
// grouped onto Hkv key/value heads (G = Hq / Hkv queries share one), attend to the P
// committed positions of the cache, to the tree tokens of earlier passes their mask
// bits allow (cache positions P .. P + T - 1) and to themselves and each other as
// the mask allows (the new keys and values, which also go into the cache at
// P + T .. P + T + M - 1 for the passes that follow).
//
// Kernel 1 (k_attn_partial): workgroup (range s, key/value head g) streams its range
// of keys in tiles of 32 through LDS (keys row-major, values transposed into the
// order the P.V product wants); wavefront t owns query rows 16t .. 16t + 15 of the
// G * M rows of head g (row = local head * M + token).  Per tile and wavefront:
//   S^T = K Q^T        16x16x32 bf16 MFMA, 2 key halves x 4 steps of 32 dimensions
//   online softmax     log2 domain; each lane holds one query's scores (4 keys per
//                      half), the row maximum takes two cross-quarter exchanges
//   O^T += V^T P^T     16x16x32 bf16 MFMA, 8 tiles of 16 dimensions; P is split
//                      into two bf16 terms (hi = bf16(p), lo = bf16(p - hi)), two
//                      MFMAs each, so the probabilities keep 16 significant bits;
//                      P is already in the B-operand layout in registers
// and writes its unnormalised partial output with the running maximum and sum.
// Kernel 1 for long ranges (k_attn_stream, eight tiles and more): its eight wavefronts take
// the tiles in turn, each for up to two tiles of query rows (with more than 32 rows two
// wavefronts share a key tile).  A wavefront keeps its own running maximum, sum and
// output, so the loop has no barrier: keys go from memory straight into the A-operand
// layout, values through a corner of LDS of its own that transposes them, and the next
// tile is loaded under the current one's softmax and P.V.  At the end the wavefronts'
// outputs are scaled to the workgroup's maximum and added in wavefront order.  Measured:
// 16450 keys of eight heads, M = 6 (17 tiles a range) 27.7 us in k_attn_partial (2.4 TB/s,
// bound by a barrier and one tile's computation after the other) against 18.4, 4180 keys
// of 16 heads (9 tiles) 23.0 against 20.4 a call; 8480 keys of four heads (5 tiles) 21.0
// against 23.3 and 2336 (3 tiles) 14.1 against 16.8, where the merge costs more than the
// tiles.
//
// Kernel 2 (k_attn_combine): one workgroup per (token, query head) combines the
// ranges in a fixed order and writes bf16; it also appends the new keys and values
// to the cache (after kernel 1, so nothing in this call reads a slot it writes).
#include <cmath>

#include "device_common.h"
#include "kernels_attn.h"

namespace subspec {

namespace {

constexpr int kAttnThreads = 256;
constexpr int kKRow = kAttnD + 8;     // bf16 per key row in LDS (16 bytes of padding)
constexpr int kVRow = kAttnTile + 8;  // bf16 per dimension row of the transposed values
constexpr int kDepth = 4;             // tiles in flight per thread

// The P.V product takes, in k-slot 8q + r of a lane in quarter q, key 4q + r (r < 4)
// and in slot 8q + 4 + r key 16 + 4q + r: exactly the keys whose scores that lane
// holds after S^T = K Q^T.  Values are stored transposed in this slot order.
__device__ __forceinline__ int value_slot(int key) {
  return key < 16 ? 8 * (key >> 2) + (key & 3) : 8 * ((key - 16) >> 2) + 4 + (key & 3);
}

struct AttnLds {
  alignas(16) uint16_t k[2][kAttnTile][kKRow];
  alignas(16) uint16_t vt[2][kAttnD][kVRow];
  alignas(16) uint32_t mask[kAttnMaskWords];
};

// Visibility of the 32 keys key0 .. key0 + 31 for one query row (bit k: key0 + k):
// committed positions (< P) always, tree positions P + j by bit j of the row's mask,
// nothing at or past k_end.  `row_mask` is the row's W words in LDS.
__device__ __forceinline__ uint32_t tile_visibility(const uint32_t* row_mask, int W, int P, int key0, int k_end) {
  uint32_t vis;
  if (key0 + kAttnTile <= P) {
    vis = ~0u;
  } else if (key0 >= P) {
    const int jb = key0 - P, w = jb >> 5, sh = jb & 31;
    const uint64_t lo = row_mask[w];
    const uint64_t hi = w + 1 < W ? row_mask[w + 1] : 0u;
    vis = static_cast<uint32_t>(((hi << 32) | lo) >> sh);
  } else {  // the tile straddles P: committed keys, then the first tree bits
    const int n = P - key0;  // 1 .. 31
    vis = (row_mask[0] << n) | ((1u << n) - 1u);
  }
  const int live = k_end - key0;  // >= 1
  return live >= kAttnTile ? vis : vis & ((1u << live) - 1u);
}

// A tile's share of one thread: two 16-byte pieces of keys (key c / 16, dimensions
// 8 (c % 16) ..) for c = thread, thread + 256, and a pair of keys' 8 dimensions of
// values (keys 2 (thread % 16) and + 1, dimensions 8 (thread / 16) ..).
struct TileRegs {
  uint4 k[2];
  uint4 v[2];
};

__device__ __forceinline__ const uint16_t* key_row(const AttnArgs& a, const uint16_t* cache,
                                                   const uint16_t* fresh, int g, int pos) {
  const int old = a.P + a.T;
  return pos < old ? cache + (static_cast<size_t>(g) * a.S + pos) * kAttnD
                   : fresh + (static_cast<size_t>(pos - old) * a.Hkv + g) * kAttnD;
}

__device__ __forceinline__ void load_tile(const AttnArgs& a, int g, int key0, int key_end, TileRegs& r) {
  const int t = threadIdx.x;
#pragma unroll
  for (int h = 0; h < 2; ++h) {
    const int c = t + h * kAttnThreads;
    const int pos = key0 + (c >> 4);
    r.k[h] = pos < key_end ? *reinterpret_cast<const uint4*>(key_row(a, a.k_cache, a.k_new, g, pos) + 8 * (c & 15))
                           : make_uint4(0, 0, 0, 0);
  }
#pragma unroll
  for (int h = 0; h < 2; ++h) {
    const int pos = key0 + 2 * (t & 15) + h;
    r.v[h] = pos < key_end ? *reinterpret_cast<const uint4*>(key_row(a, a.v_cache, a.v_new, g, pos) + 8 * (t >> 4))
                           : make_uint4(0, 0, 0, 0);
  }
}

__device__ __forceinline__ void store_tile(AttnLds& L, int buf, const TileRegs& r) {
  const int t = threadIdx.x;
#pragma unroll
  for (int h = 0; h < 2; ++h) {
    const int c = t + h * kAttnThreads;
    *reinterpret_cast<uint4*>(&L.k[buf][c >> 4][8 * (c & 15)]) = r.k[h];
  }
  // two keys (adjacent slots) of one dimension per 32-bit word
  const int slot = value_slot(2 * (t & 15));
  const int d0 = 8 * (t >> 4);
  const uint32_t a0[4] = {r.v[0].x, r.v[0].y, r.v[0].z, r.v[0].w};
  const uint32_t a1[4] = {r.v[1].x, r.v[1].y, r.v[1].z, r.v[1].w};
#pragma unroll
  for (int e = 0; e < 4; ++e) {
    const uint32_t lo = __builtin_amdgcn_perm(a1[e], a0[e], 0x05040100u);  // dimension 2e: key, key + 1
    const uint32_t hi = __builtin_amdgcn_perm(a1[e], a0[e], 0x07060302u);  // dimension 2e + 1
    *reinterpret_cast<uint32_t*>(&L.vt[buf][d0 + 2 * e][slot]) = lo;
    *reinterpret_cast<uint32_t*>(&L.vt[buf][d0 + 2 * e + 1][slot]) = hi;
  }
}

__device__ __forceinline__ uint32_t pack_bf16(float lo, float hi) {
  return static_cast<uint32_t>(float_to_bf16_bits(lo)) | (static_cast<uint32_t>(float_to_bf16_bits(hi)) << 16);
}

__device__ __forceinline__ float bf16_lo(uint32_t w) { return __uint_as_float(w << 16); }
__device__ __forceinline__ float bf16_hi(uint32_t w) { return __uint_as_float(w & 0xFFFF0000u); }

template <int QT>
__global__ __launch_bounds__(kAttnThreads) void k_attn_partial(AttnArgs a) {
  __shared__ AttnLds L;
  const int s = blockIdx.x, g = blockIdx.y;
  const int lane = threadIdx.x % kWave, wave = threadIdx.x / kWave;
  const int col = lane & 15, quarter = lane >> 4;
  const int G = a.Hq / a.Hkv;
  const int rows = G * a.M;
  const int Ltot = a.P + a.T + a.M;
  const int k_begin = s * a.tiles_per_split * kAttnTile;
  const int k_end = min(Ltot, k_begin + a.tiles_per_split * kAttnTile);
  const int ntiles = (k_end - k_begin + kAttnTile - 1) / kAttnTile;

  // this lane's query row (one per lane and wavefront) and its fragments of q
  const int row = 16 * wave + col;
  const bool live_row = wave < QT && row < rows;
  const int qi = live_row ? row % a.M : 0;
  const int hl = live_row ? row / a.M : 0;
  bf16x8_t qf[4];
#pragma unroll
  for (int j = 0; j < 4; ++j) {
    uint4 w = make_uint4(0, 0, 0, 0);
    if (live_row)
      w = *reinterpret_cast<const uint4*>(a.q + (static_cast<size_t>(qi) * a.Hq + g * G + hl) * kAttnD + 32 * j +
                                          8 * quarter);
    qf[j] = __builtin_bit_cast(bf16x8_t, w);
  }
  for (int w = threadIdx.x; w < a.M * a.W; w += kAttnThreads) L.mask[w] = a.mask[w];

  float m = -INFINITY, lsum = 0.f;
  f32x4_t o[8];
#pragma unroll
  for (int dt = 0; dt < 8; ++dt) o[dt] = f32x4_t{0.f, 0.f, 0.f, 0.f};

  TileRegs ring[kDepth];
#pragma unroll
  for (int d = 0; d < kDepth; ++d)
    if (d < ntiles) load_tile(a, g, k_begin + d * kAttnTile, k_end, ring[d]);

  for (int n0 = 0; n0 < ntiles; n0 += kDepth) {
#pragma unroll
    for (int d = 0; d < kDepth; ++d) {
      const int n = n0 + d;
      if (n >= ntiles) break;
      const int buf = n & 1;
      // buffer buf was last read two tiles ago, before the previous barrier
      store_tile(L, buf, ring[d]);
      if (n + kDepth < ntiles) load_tile(a, g, k_begin + (n + kDepth) * kAttnTile, k_end, ring[d]);
      __syncthreads();
      if (wave < QT) {
        const int key0 = k_begin + n * kAttnTile;
        // S^T = K Q^T: lane holds keys 16u + 4 quarter + r of its query
        f32x4_t st[2];
#pragma unroll
        for (int u = 0; u < 2; ++u) {
          st[u] = f32x4_t{0.f, 0.f, 0.f, 0.f};
#pragma unroll
          for (int j = 0; j < 4; ++j) {
            const bf16x8_t kf = *reinterpret_cast<const bf16x8_t*>(&L.k[buf][16 * u + col][32 * j + 8 * quarter]);
            st[u] = __builtin_amdgcn_mfma_f32_16x16x32_bf16(kf, qf[j], st[u], 0, 0, 0);
          }
        }
        // scale, mask (committed positions are always visible), online softmax
        const uint32_t vis = live_row ? tile_visibility(&L.mask[qi * a.W], a.W, a.P, key0, k_end) : 0u;
        float sv[2][4];
        float mx = -INFINITY;
#pragma unroll
        for (int u = 0; u < 2; ++u)
#pragma unroll
          for (int r = 0; r < 4; ++r) {
            const bool ok = (vis >> (16 * u + 4 * quarter + r)) & 1u;
            sv[u][r] = ok ? st[u][r] * a.scale_log2 : -INFINITY;
            mx = fmaxf(mx, sv[u][r]);
          }
        mx = fmaxf(mx, __shfl_xor(mx, 16));
        mx = fmaxf(mx, __shfl_xor(mx, 32));
        const float mn = fmaxf(m, mx);
        // raw 2^x (a probability below 2^-126 flushing to zero does not matter)
        const float alpha = m == -INFINITY ? 0.f : __builtin_amdgcn_exp2f(m - mn);
        // p = hi + lo in bf16; the same two terms feed P.V and the sum
        uint32_t ph[4], pl[4];
        float add = 0.f;
#pragma unroll
        for (int u = 0; u < 2; ++u)
#pragma unroll
          for (int r = 0; r < 4; r += 2) {
            const float p0 = sv[u][r] == -INFINITY ? 0.f : __builtin_amdgcn_exp2f(sv[u][r] - mn);
            const float p1 = sv[u][r + 1] == -INFINITY ? 0.f : __builtin_amdgcn_exp2f(sv[u][r + 1] - mn);
            const uint32_t h = pack_bf16(p0, p1);
            const uint32_t l = pack_bf16(p0 - bf16_lo(h), p1 - bf16_hi(h));
            ph[2 * u + r / 2] = h;
            pl[2 * u + r / 2] = l;
            add += (bf16_lo(h) + bf16_lo(l)) + (bf16_hi(h) + bf16_hi(l));
          }
        lsum = lsum * alpha + add;
        m = mn;
        const bf16x8_t pfh = __builtin_bit_cast(bf16x8_t, make_uint4(ph[0], ph[1], ph[2], ph[3]));
        const bf16x8_t pfl = __builtin_bit_cast(bf16x8_t, make_uint4(pl[0], pl[1], pl[2], pl[3]));
        if (__builtin_amdgcn_ballot_w64(alpha != 1.f)) {  // some row's maximum moved
#pragma unroll
          for (int dt = 0; dt < 8; ++dt) o[dt] *= alpha;
        }
#pragma unroll
        for (int dt = 0; dt < 8; ++dt) {
          const bf16x8_t vf = *reinterpret_cast<const bf16x8_t*>(&L.vt[buf][16 * dt + col][8 * quarter]);
          o[dt] = __builtin_amdgcn_mfma_f32_16x16x32_bf16(vf, pfh, o[dt], 0, 0, 0);
          o[dt] = __builtin_amdgcn_mfma_f32_16x16x32_bf16(vf, pfl, o[dt], 0, 0, 0);
        }
      }
    }
  }

  if (wave < QT) {
    // the four quarters hold partial sums of the same query
    lsum += __shfl_xor(lsum, 16);
    lsum += __shfl_xor(lsum, 32);
  }
  if (live_row) {  // padding rows are never read
    const size_t base = (static_cast<size_t>(g) * a.splits + s) * a.rows_pad + row;
#pragma unroll
    for (int dt = 0; dt < 8; ++dt)
      *reinterpret_cast<f32x4_t*>(a.part_o + base * kAttnD + 16 * dt + 4 * quarter) = o[dt];
    if (quarter == 0) {
      a.part_ml[2 * base] = m;
      a.part_ml[2 * base + 1] = lsum;
    }
  }
}

constexpr int kStreamWaves = 8;
constexpr int kStreamThreads = kStreamWaves * kWave;
constexpr int kStreamTiles = 8;        // tiles per range from which k_attn_stream is taken
constexpr int kMergeRow = kAttnD + 4;  // floats per query row of a wavefront's merged output

union alignas(16) WaveLds {
  uint16_t vt[kAttnD][kVRow];  // a wavefront's values, transposed
  float o[16][kMergeRow];      // its output of one query tile
};

struct StreamLds {
  WaveLds w[kStreamWaves];
  float m[kStreamWaves][32], l[kStreamWaves][32];  // its maxima and sums per query row
  alignas(16) uint32_t mask[kAttnMaskWords];
};

// One lane's share of a tile.  Keys: A-operand fragments, key 16u + lane % 16, dimensions
// 32j + 8 (lane / 16) .. + 7.  Values: keys 2 (lane % 16) + h, dimensions
// 32j + 8 (lane / 16) .. + 7.
struct StreamRegs {
  uint4 k[2][4];
  uint4 v[4][2];
};

__device__ __forceinline__ void stream_load(const AttnArgs& a, int g, int key0, int key_end, int lane, StreamRegs& r) {
  const int col = lane & 15, d0 = 8 * (lane >> 4);
#pragma unroll
  for (int u = 0; u < 2; ++u) {
    // keys past the range repeat its last one (masked below)
    const uint16_t* row = key_row(a, a.k_cache, a.k_new, g, min(key0 + 16 * u + col, key_end - 1)) + d0;
#pragma unroll
    for (int j = 0; j < 4; ++j) r.k[u][j] = *reinterpret_cast<const uint4*>(row + 32 * j);
  }
#pragma unroll
  for (int h = 0; h < 2; ++h) {
    const uint16_t* row = key_row(a, a.v_cache, a.v_new, g, min(key0 + 2 * col + h, key_end - 1)) + d0;
#pragma unroll
    for (int j = 0; j < 4; ++j) r.v[j][h] = *reinterpret_cast<const uint4*>(row + 32 * j);
  }
}

// Values of keys at and past `live` become zeros: their probability is zero, and zero times
// an infinite value (the repeated last key's) would be NaN.
__device__ __forceinline__ void zero_values(StreamRegs& r, int live, int lane) {
#pragma unroll
  for (int h = 0; h < 2; ++h)
    if (2 * (lane & 15) + h >= live) {
#pragma unroll
      for (int j = 0; j < 4; ++j) r.v[j][h] = make_uint4(0, 0, 0, 0);
    }
}

__device__ __forceinline__ void store_values(uint16_t (&vt)[kAttnD][kVRow], const StreamRegs& r, int lane) {
  // two keys (adjacent slots) of one dimension per 32-bit word
  const int slot = value_slot(2 * (lane & 15));
#pragma unroll
  for (int j = 0; j < 4; ++j) {
    const int d0 = 32 * j + 8 * (lane >> 4);
    const uint32_t a0[4] = {r.v[j][0].x, r.v[j][0].y, r.v[j][0].z, r.v[j][0].w};
    const uint32_t a1[4] = {r.v[j][1].x, r.v[j][1].y, r.v[j][1].z, r.v[j][1].w};
#pragma unroll
    for (int e = 0; e < 4; ++e) {
      const uint32_t lo = __builtin_amdgcn_perm(a1[e], a0[e], 0x05040100u);  // dimension 2e: key, key + 1
      const uint32_t hi = __builtin_amdgcn_perm(a1[e], a0[e], 0x07060302u);  // dimension 2e + 1
      *reinterpret_cast<uint32_t*>(&vt[d0 + 2 * e][slot]) = lo;
      *reinterpret_cast<uint32_t*>(&vt[d0 + 2 * e + 1][slot]) = hi;
    }
  }
}

// Orders LDS accesses of a wavefront's lanes to each other's words, for the compiler (the
// hardware keeps a wavefront's LDS operations in order; no instruction is emitted).
__device__ __forceinline__ void wave_lds_fence() {
  __builtin_amdgcn_fence(__ATOMIC_RELEASE, "wavefront");
  __builtin_amdgcn_wave_barrier();
  __builtin_amdgcn_fence(__ATOMIC_ACQUIRE, "wavefront");
}

// QT: query tiles of 16 rows (1 .. 4); a wavefront takes QW of them.
template <int QT>
__global__ __launch_bounds__(kStreamThreads) __attribute__((amdgpu_waves_per_eu(2))) void k_attn_stream(AttnArgs a) {
  constexpr int QW = QT < 2 ? 1 : 2;
  constexpr int QG = (QT + 1) / 2;            // wavefronts that share a key tile
  constexpr int KW = kStreamWaves / QG;         // key tiles at a time
  __shared__ StreamLds L;
  const int s = blockIdx.x, g = blockIdx.y;
  const int lane = threadIdx.x % kWave;
  const int wave = __builtin_amdgcn_readfirstlane(static_cast<int>(threadIdx.x / kWave));
  const int qg = wave % QG, kw = wave / QG;
  const int col = lane & 15, quarter = lane >> 4;
  const int G = a.Hq / a.Hkv;
  const int rows = G * a.M;
  const int Ltot = a.P + a.T + a.M;
  const int k_begin = s * a.tiles_per_split * kAttnTile;
  const int k_end = min(Ltot, k_begin + a.tiles_per_split * kAttnTile);
  const int ntiles = (k_end - k_begin + kAttnTile - 1) / kAttnTile;

  StreamRegs r;
  if (kw < ntiles) stream_load(a, g, k_begin + kw * kAttnTile, k_end, lane, r);

  // this lane's query row in each of the wavefront's query tiles, and its fragments of q
  bool live[QW];
  int qi[QW];
  bf16x8_t qf[QW][4];
#pragma unroll
  for (int t = 0; t < QW; ++t) {
    const int row = 16 * (QW * qg + t) + col;
    live[t] = row < rows;
    qi[t] = live[t] ? row % a.M : 0;
    const int hl = live[t] ? row / a.M : 0;
#pragma unroll
    for (int j = 0; j < 4; ++j) {
      uint4 w = make_uint4(0, 0, 0, 0);
      if (live[t])
        w = *reinterpret_cast<const uint4*>(a.q + (static_cast<size_t>(qi[t]) * a.Hq + g * G + hl) * kAttnD + 32 * j +
                                            8 * quarter);
      qf[t][j] = __builtin_bit_cast(bf16x8_t, w);
    }
  }
  for (int w = threadIdx.x; w < a.M * a.W; w += kStreamThreads) L.mask[w] = a.mask[w];
  __syncthreads();

  float m[QW], lsum[QW];
  f32x4_t o[QW][8];
#pragma unroll
  for (int t = 0; t < QW; ++t) {
    m[t] = -INFINITY;
    lsum[t] = 0.f;
#pragma unroll
    for (int dt = 0; dt < 8; ++dt) o[t][dt] = f32x4_t{0.f, 0.f, 0.f, 0.f};
  }
  auto& vt = L.w[wave].vt;
  for (int n = kw; n < ntiles; n += KW) {
    const int key0 = k_begin + n * kAttnTile;
    if (key0 + kAttnTile > k_end) zero_values(r, k_end - key0, lane);
    store_values(vt, r, lane);
    wave_lds_fence();  // the products below read other lanes' words
    // S^T = K Q^T: lane holds keys 16u + 4 quarter + r of its query
    f32x4_t st[QW][2];
#pragma unroll
    for (int u = 0; u < 2; ++u)
#pragma unroll
      for (int j = 0; j < 4; ++j) {
        const bf16x8_t kf = __builtin_bit_cast(bf16x8_t, r.k[u][j]);
#pragma unroll
        for (int t = 0; t < QW; ++t)
          st[t][u] = __builtin_amdgcn_mfma_f32_16x16x32_bf16(kf, qf[t][j], j == 0 ? f32x4_t{0.f, 0.f, 0.f, 0.f} : st[t][u],
                                                             0, 0, 0);
      }
    if (n + KW < ntiles) stream_load(a, g, k_begin + (n + KW) * kAttnTile, k_end, lane, r);
    bf16x8_t pfh[QW], pfl[QW];
#pragma unroll
    for (int t = 0; t < QW; ++t) {
      // scale, mask (committed positions are always visible), online softmax
      const uint32_t vis = live[t] ? tile_visibility(&L.mask[qi[t] * a.W], a.W, a.P, key0, k_end) : 0u;
      float sv[2][4];
      float mx = -INFINITY;
#pragma unroll
      for (int u = 0; u < 2; ++u)
#pragma unroll
        for (int e = 0; e < 4; ++e) {
          const bool ok = (vis >> (16 * u + 4 * quarter + e)) & 1u;
          const float sc = st[t][u][e];
          sv[u][e] = ok ? sc * a.scale_log2 : -INFINITY;
          mx = fmaxf(mx, sv[u][e]);
        }
      mx = fmaxf(mx, __shfl_xor(mx, 16));
      mx = fmaxf(mx, __shfl_xor(mx, 32));
      const float mn = fmaxf(m[t], mx);
      // raw 2^x (a probability below 2^-126 flushing to zero does not matter)
      const float alpha = m[t] == -INFINITY ? 0.f : __builtin_amdgcn_exp2f(m[t] - mn);
      // p = hi + lo in bf16; the same two terms feed P.V and the sum
      uint32_t ph[4], pl[4];
      float add = 0.f;
#pragma unroll
      for (int u = 0; u < 2; ++u)
#pragma unroll
        for (int e = 0; e < 4; e += 2) {
          const float p0 = sv[u][e] == -INFINITY ? 0.f : __builtin_amdgcn_exp2f(sv[u][e] - mn);
          const float p1 = sv[u][e + 1] == -INFINITY ? 0.f : __builtin_amdgcn_exp2f(sv[u][e + 1] - mn);
          const uint32_t h = pack_bf16(p0, p1);
          const uint32_t l = pack_bf16(p0 - bf16_lo(h), p1 - bf16_hi(h));
          ph[2 * u + e / 2] = h;
          pl[2 * u + e / 2] = l;
          add += (bf16_lo(h) + bf16_lo(l)) + (bf16_hi(h) + bf16_hi(l));
        }
      lsum[t] = lsum[t] * alpha + add;
      m[t] = mn;
      pfh[t] = __builtin_bit_cast(bf16x8_t, make_uint4(ph[0], ph[1], ph[2], ph[3]));
      pfl[t] = __builtin_bit_cast(bf16x8_t, make_uint4(pl[0], pl[1], pl[2], pl[3]));
      if (__builtin_amdgcn_ballot_w64(alpha != 1.f)) {  // some row's maximum moved
#pragma unroll
        for (int dt = 0; dt < 8; ++dt) o[t][dt] *= alpha;
      }
    }
#pragma unroll
    for (int dt = 0; dt < 8; ++dt) {
      const bf16x8_t vf = *reinterpret_cast<const bf16x8_t*>(&vt[16 * dt + col][8 * quarter]);
#pragma unroll
      for (int t = 0; t < QW; ++t) {
        o[t][dt] = __builtin_amdgcn_mfma_f32_16x16x32_bf16(vf, pfh[t], o[t][dt], 0, 0, 0);
        o[t][dt] = __builtin_amdgcn_mfma_f32_16x16x32_bf16(vf, pfl[t], o[t][dt], 0, 0, 0);
      }
    }
    wave_lds_fence();  // the next stores overwrite what other lanes read
  }

  // The workgroup's maximum per row; every wavefront scales its output and sum to it.
#pragma unroll
  for (int t = 0; t < QW; ++t) {
    // the four quarters hold partial sums of the same query
    lsum[t] += __shfl_xor(lsum[t], 16);
    lsum[t] += __shfl_xor(lsum[t], 32);
    if (quarter == 0) L.m[wave][16 * t + col] = m[t];
  }
  __syncthreads();
  float mall[QW];
#pragma unroll
  for (int t = 0; t < QW; ++t) {
    mall[t] = -INFINITY;
#pragma unroll
    for (int w = 0; w < KW; ++w) mall[t] = fmaxf(mall[t], L.m[w * QG + qg][16 * t + col]);
    const float sc = m[t] == -INFINITY ? 0.f : __builtin_amdgcn_exp2f(m[t] - mall[t]);
#pragma unroll
    for (int dt = 0; dt < 8; ++dt) o[t][dt] *= sc;
    if (quarter == 0) L.l[wave][16 * t + col] = lsum[t] * sc;
  }
  // One query tile of every wavefront at a time: outputs [row][dimension] in LDS, then the
  // workgroup adds the wavefronts' in order, four dimensions a thread.
#pragma unroll
  for (int t = 0; t < QW; ++t) {
#pragma unroll
    for (int dt = 0; dt < 8; ++dt)
      *reinterpret_cast<f32x4_t*>(&L.w[wave].o[col][16 * dt + 4 * quarter]) = o[t][dt];
    __syncthreads();
    for (int i = threadIdx.x; i < QG * 16 * (kAttnD / 4); i += kStreamThreads) {
      const int qw = i / (16 * (kAttnD / 4)), rr = i / (kAttnD / 4) % 16, d4 = 4 * (i % (kAttnD / 4));
      const int row = 16 * (QW * qw + t) + rr;
      if (row >= rows) continue;  // padding rows are never read
      f32x4_t sum = *reinterpret_cast<const f32x4_t*>(&L.w[qw].o[rr][d4]);
#pragma unroll
      for (int w = 1; w < KW; ++w) sum += *reinterpret_cast<const f32x4_t*>(&L.w[w * QG + qw].o[rr][d4]);
      const size_t base = (static_cast<size_t>(g) * a.splits + s) * a.rows_pad + row;
      *reinterpret_cast<f32x4_t*>(a.part_o + base * kAttnD + d4) = sum;
      if (d4 == 0) {
        float mm = -INFINITY, ls = 0.f;
#pragma unroll
        for (int w = 0; w < KW; ++w) {
          mm = fmaxf(mm, L.m[w * QG + qw][16 * t + rr]);
          ls += L.l[w * QG + qw][16 * t + rr];
        }
        a.part_ml[2 * base] = mm;
        a.part_ml[2 * base + 1] = ls;
      }
    }
    if (t + 1 < QW) __syncthreads();
  }
}

// One workgroup per (token i, query head h), one thread per dimension.  The first kBatch
// ranges' outputs are requested together with the (max, sum) pairs, so the usual call waits
// for memory once; each pair is turned into a weight by one thread, and the outputs are
// summed in range order.  Later ranges come kMore at a time: a second batch of 32 for the
// 33 to 48 ranges of 3000 to 4400 keys of four heads took 15.2 us a call, one of 16 14.1
// (batches of 16 throughout, none requested early: 14.8).
__global__ __launch_bounds__(kAttnD) void k_attn_combine(AttnArgs a) {
  __shared__ float sm[kAttnMaxSplits], sl[kAttnMaxSplits];
  constexpr int kBatch = 32, kMore = 16;  // requested at the start, and at a time after those
  const int i = blockIdx.x / a.Hq, h = blockIdx.x % a.Hq;
  const int d = threadIdx.x;
  const int G = a.Hq / a.Hkv;
  const int g = h / G, hl = h % G;
  const int row = hl * a.M + i;
  const int ns = a.splits;
  const size_t base = static_cast<size_t>(g) * ns * a.rows_pad + row;
  const float* po = a.part_o + base * kAttnD + d;
  const size_t step = static_cast<size_t>(a.rows_pad) * kAttnD;
  for (int s = d; s < ns; s += kAttnD) {
    const float2 ml = *reinterpret_cast<const float2*>(a.part_ml + 2 * (base + static_cast<size_t>(s) * a.rows_pad));
    sm[s] = ml.x;
    sl[s] = ml.y;
  }
  float v[kBatch];
#pragma unroll
  for (int u = 0; u < kBatch; ++u) v[u] = u < ns ? po[u * step] : 0.f;
  __syncthreads();
  float mmax = -INFINITY;
  for (int s = 0; s < ns; ++s) mmax = fmaxf(mmax, sm[s]);
  __syncthreads();
  for (int s = d; s < ns; s += kAttnD) sm[s] = sm[s] == -INFINITY ? 0.f : exp2f(sm[s] - mmax);
  __syncthreads();
  float den = 0.f, num = 0.f;
#pragma unroll
  for (int u = 0; u < kBatch; ++u)
    if (u < ns) {
      den += sm[u] * sl[u];
      num += sm[u] * v[u];
    }
  for (int s0 = kBatch; s0 < ns; s0 += kMore) {
#pragma unroll
    for (int u = 0; u < kMore; ++u) v[u] = s0 + u < ns ? po[(s0 + u) * step] : 0.f;
#pragma unroll
    for (int u = 0; u < kMore; ++u)
      if (s0 + u < ns) {
        den += sm[s0 + u] * sl[s0 + u];
        num += sm[s0 + u] * v[u];
      }
  }
  a.out[(static_cast<size_t>(i) * a.Hq + h) * kAttnD + d] = float_to_bf16_bits(den > 0.f ? num / den : 0.f);
  // append this token's key and value for head g (once per key/value head)
  if (hl == 0) {
    const size_t dst = (static_cast<size_t>(g) * a.S + a.P + a.T + i) * kAttnD + d;
    const size_t src = (static_cast<size_t>(i) * a.Hkv + g) * kAttnD + d;
    a.k_cache[dst] = a.k_new[src];
    a.v_cache[dst] = a.v_new[src];
  }
}

}  // namespace

void attn_plan(int M, int Hq, int Hkv, int P, int T, int* splits, int* tiles_per_split) {
  (void)Hq;
  const int L = P + T + M;
  const int tiles = (L + kAttnTile - 1) / kAttnTile;
  // at most one workgroup per CU of the 256 and at least three tiles each (all in
  // flight at once): fewer, longer ranges keep the partial outputs small beside the
  // keys and values read (three measured fastest at 2336 keys; two and four were
  // within 4 %, six 20 % slower)
  constexpr int kMinTiles = 3;
  int tps = (tiles * Hkv + 255) / 256;
  if (tps < kMinTiles) tps = kMinTiles;
  if (tps > tiles) tps = tiles;
  *tiles_per_split = tps;
  *splits = (tiles + tps - 1) / tps;
}

size_t attn_workspace_bytes(int M, int Hq, int Hkv, int P, int T) {
  int splits = 0, tps = 0;
  attn_plan(M, Hq, Hkv, P, T, &splits, &tps);
  const int rows_pad = 16 * ((Hq / Hkv * M + 15) / 16);
  const size_t n = static_cast<size_t>(Hkv) * splits * rows_pad;
  // The partials follow the split-K completion counters at the workspace's start.
  return kSplitCounterBytes + n * kAttnD * sizeof(float) + n * 2 * sizeof(float);
}

hipError_t launch_tree_attention(const AttnArgs& a, hipStream_t st) {
  const dim3 grid(a.splits, a.Hkv), block(kAttnThreads), wide(kStreamThreads);
  const bool stream = a.tiles_per_split >= kStreamTiles;
  if (stream) switch (a.rows_pad / 16) {
    case 1: hipLaunchKernelGGL(k_attn_stream<1>, grid, wide, 0, st, a); break;
    case 2: hipLaunchKernelGGL(k_attn_stream<2>, grid, wide, 0, st, a); break;
    case 3: hipLaunchKernelGGL(k_attn_stream<3>, grid, wide, 0, st, a); break;
    default: hipLaunchKernelGGL(k_attn_stream<4>, grid, wide, 0, st, a); break;
  }
  else switch (a.rows_pad / 16) {
    case 1: hipLaunchKernelGGL(k_attn_partial<1>, grid, block, 0, st, a); break;
    case 2: hipLaunchKernelGGL(k_attn_partial<2>, grid, block, 0, st, a); break;
    case 3: hipLaunchKernelGGL(k_attn_partial<3>, grid, block, 0, st, a); break;
    default: hipLaunchKernelGGL(k_attn_partial<4>, grid, block, 0, st, a); break;
  }
  hipError_t e = hipGetLastError();
  if (e != hipSuccess) return e;
  hipLaunchKernelGGL(k_attn_combine, dim3(a.M * a.Hq), dim3(kAttnD), 0, st, a);
  return hipGetLastError();
}

}  // namespace subspec
