// Draft-tree expansion with probability sharpening (SubSpec Sec. 4.2 and App. D).
//
// In each draft pass every leaf i of the tree yields logits l_i over the vocabulary.
// A candidate (i, v) scores  s_i + log softmax(l_i / T)(v)  -- the logarithm of the
// product of the parent's path score and the sharpened conditional probability --
// and the k best candidates over all leaves become the next leaves.  Order: larger
// score first, then the smaller flat index i * V + v.
//
// One launch, two phases.  Workgroup (row i, chunk c) streams its slice of l_i once
// (16-byte loads of eight bf16 logits, four loads in flight per thread), keeping per thread an online softmax pair
// (running max m, sum of exp(z - m)) and a sorted list of its k best z = l / T; the
// workgroup merges both and stores them.  The last workgroup to finish (completion
// counter, as in the qlinear split-K) combines the pairs of each row into its
// log-sum-exp, turns every stored candidate into a score and selects the k best.
// Every reduction runs in a fixed order, so results are bit-reproducible.
//
// What bounds it is the chain of latencies of the two phases, not the logits: of 20.2 us
// at R = 6, V = 152064, k = 6 with 450 workgroups, 2.2 were the launch, 3.0 the logits, 3.5
// the workgroup's selection, 4.1 the completion and 7.4 the second phase.  So no more
// workgroups run than the second phase's threads hold lists (256 up to 32 rows; tree_plan),
// the lists arrive in the second phase's registers with one wait, and
// the reductions stay in DPP moves.
#include <climits>
#include <cmath>

#include "device_common.h"
#include "kernels_tree.h"

namespace subspec {

namespace {

constexpr int kTreeThreads = 256;
constexpr int kTreeWaves = kTreeThreads / kWave;
constexpr int kTreeMaxBlocks = 1024;  // R * chunks never exceeds this (tree_plan)
constexpr int kTreeLoads = 4;         // logit loads in flight per thread
constexpr int kTreeCoherent = 16;     // sc1: coherent at agent scope
constexpr int kTreeCap = 2048;        // candidates ranked at once in LDS

// Candidate order: larger value first, then smaller index.
__device__ __forceinline__ bool better(float av, int ai, float bv, int bi) {
  return av > bv || (av == bv && ai < bi);
}

// A thread's KMAX best candidates, best first; empty slots hold (-inf, INT_MAX).
template <int KMAX>
struct TopList {
  float v[KMAX];
  int i[KMAX];
  __device__ __forceinline__ void clear() {
#pragma unroll
    for (int j = 0; j < KMAX; ++j) {
      v[j] = -INFINITY;
      i[j] = INT_MAX;
    }
  }
  // One pass of compare-exchange down the list keeps it sorted.
  __device__ __forceinline__ void insert(float val, int idx) {
#pragma unroll
    for (int j = 0; j < KMAX; ++j) {
      const bool b = better(val, idx, v[j], i[j]);
      const float tv = v[j];
      const int ti = i[j];
      v[j] = b ? val : tv;
      i[j] = b ? idx : ti;
      val = b ? tv : val;
      idx = b ? ti : idx;
    }
  }
  __device__ __forceinline__ void pop() {
#pragma unroll
    for (int j = 0; j + 1 < KMAX; ++j) {
      v[j] = v[j + 1];
      i[j] = i[j + 1];
    }
    v[KMAX - 1] = -INFINITY;
    i[KMAX - 1] = INT_MAX;
  }
};

// (m, s) pairs of an online softmax: s = sum of exp(z - m) over the values seen.
__device__ __forceinline__ void softmax_merge(float& m, float& s, float m2, float s2) {
  if (m2 > m) {
    const float t = m;
    m = m2;
    m2 = t;
    const float u = s;
    s = s2;
    s2 = u;
  }
  if (m2 != -INFINITY) s += s2 * __expf(m2 - m);
}

struct TreeShared {
  float wm[kTreeWaves], ws[kTreeWaves];
  // per-wavefront heads of a selection round; rounds alternate between the two
  // slots, so one barrier per round suffices
  float bv[2][kTreeWaves];
  int bi[2][kTreeWaves];
  int last;
  int n;  // candidates appended to the LDS buffer
  // the k winners of the workgroup, stored to memory after the last round (a store
  // inside a round would make every following barrier wait for it)
  float win_v[kTreeMaxK];
  int win_i[kTreeMaxK];
};

// One step of a wavefront reduction over (value, index) with a DPP lane move.  Rows
// outside ROW_MASK keep their own pair (the move returns it as `old`).
template <int CTRL, int ROW_MASK>
__device__ __forceinline__ void dpp_best(float& v, int& i) {
  const int vb = __builtin_bit_cast(int, v);
  const float ov = __builtin_bit_cast(float, __builtin_amdgcn_update_dpp(vb, vb, CTRL, ROW_MASK, 0xF, false));
  const int oi = __builtin_amdgcn_update_dpp(i, i, CTRL, ROW_MASK, 0xF, false);
  if (better(ov, oi, v, i)) {
    v = ov;
    i = oi;
  }
}

// The wavefront's best (value, index) in every lane: quads, half rows and rows by
// lane permutations, then rows 0-1 and 2-3 by row broadcasts into lane 63.
__device__ __forceinline__ void wave_best(float& v, int& i) {
  dpp_best<0xB1, 0xF>(v, i);   // quad_perm [1,0,3,2]
  dpp_best<0x4E, 0xF>(v, i);   // quad_perm [2,3,0,1]
  dpp_best<0x141, 0xF>(v, i);  // row_half_mirror
  dpp_best<0x140, 0xF>(v, i);  // row_mirror
  dpp_best<0x142, 0xA>(v, i);  // row_bcast:15 into rows 1 and 3
  dpp_best<0x143, 0xC>(v, i);  // row_bcast:31 into rows 2 and 3
  v = __builtin_bit_cast(float, __builtin_amdgcn_readlane(__builtin_bit_cast(int, v), kWave - 1));
  i = __builtin_amdgcn_readlane(i, kWave - 1);
}

// Largest value over the wavefront (same lane moves), in every lane.
template <int CTRL, int ROW_MASK>
__device__ __forceinline__ float dpp_max_step(float v) {
  const int vb = __builtin_bit_cast(int, v);
  return fmaxf(v, __builtin_bit_cast(float, __builtin_amdgcn_update_dpp(vb, vb, CTRL, ROW_MASK, 0xF, false)));
}
__device__ __forceinline__ float wave_max(float v) {
  v = dpp_max_step<0xB1, 0xF>(v);
  v = dpp_max_step<0x4E, 0xF>(v);
  v = dpp_max_step<0x141, 0xF>(v);
  v = dpp_max_step<0x140, 0xF>(v);
  v = dpp_max_step<0x142, 0xA>(v);
  v = dpp_max_step<0x143, 0xC>(v);
  return __builtin_bit_cast(float, __builtin_amdgcn_readlane(__builtin_bit_cast(int, v), kWave - 1));
}

// Sum over the wavefront (same lane moves; rows that take no part add nothing), in every lane.
template <int CTRL, int ROW_MASK>
__device__ __forceinline__ float dpp_sum_step(float v) {
  return v + __builtin_bit_cast(float, __builtin_amdgcn_update_dpp(0, __builtin_bit_cast(int, v), CTRL, ROW_MASK, 0xF, false));
}
__device__ __forceinline__ float wave_sum(float v) {
  v = dpp_sum_step<0xB1, 0xF>(v);
  v = dpp_sum_step<0x4E, 0xF>(v);
  v = dpp_sum_step<0x141, 0xF>(v);
  v = dpp_sum_step<0x140, 0xF>(v);
  v = dpp_sum_step<0x142, 0xA>(v);
  v = dpp_sum_step<0x143, 0xC>(v);
  return __builtin_bit_cast(float, __builtin_amdgcn_readlane(__builtin_bit_cast(int, v), kWave - 1));
}

// Workgroup-wide best head of the threads' lists, removed from its owner; rounds
// 0..k-1 give the workgroup's k best in order.  All threads get (value, index).
// A thread can write the slot of round j + 2 only after every thread has reached
// the barrier of round j + 1, i.e. has finished reading round j.
template <int KMAX>
__device__ __forceinline__ void take_best(TopList<KMAX>& t, TreeShared& sh, int round, float& val, int& idx) {
  float v = t.v[0];
  int i = t.i[0];
  wave_best(v, i);
  const int lane = threadIdx.x % kWave, wave = threadIdx.x / kWave;
  const int slot = round & 1;
  if (lane == 0) {
    sh.bv[slot][wave] = v;
    sh.bi[slot][wave] = i;
  }
  __syncthreads();
  val = sh.bv[slot][0];
  idx = sh.bi[slot][0];
#pragma unroll
  for (int w = 1; w < kTreeWaves; ++w)
    if (better(sh.bv[slot][w], sh.bi[slot][w], val, idx)) {
      val = sh.bv[slot][w];
      idx = sh.bi[slot][w];
    }
  if (t.i[0] == idx) t.pop();
}

// A value that at least k of the lanes' heads reach: the largest heads are taken off
// round by round (tied lanes together) until k are counted; -inf if the wavefront
// holds fewer than k finite heads.  Called with every lane active.
__device__ __forceinline__ float wave_kth_head(float h, int k) {
  float th = -INFINITY;
  if (k > 8) {
    // Many rounds: the bound from its top 16 bits instead (any value that k heads reach
    // will do), found bit by bit in the order-preserving integer form of a float.
    if (__popcll(__ballot(h > -INFINITY)) < k) return th;
    const uint32_t b = __float_as_uint(h);
    const uint32_t u = b & 0x80000000u ? ~b : b | 0x80000000u;
    uint32_t t = 0;
#pragma unroll
    for (int bit = 31; bit >= 16; --bit) {
      const uint32_t c = t | (1u << bit);
      if (__popcll(__ballot(u >= c)) >= k) t = c;
    }
    const float f = __uint_as_float(t & 0x80000000u ? t ^ 0x80000000u : ~t);
    return f == f ? f : -INFINITY;  // a prefix below every number is no bound
  }
  int cnt = 0;
  while (cnt < k) {
    const float mx = wave_max(h);
    if (mx == -INFINITY) return -INFINITY;
    cnt += __popcll(__ballot(h == mx));
    th = mx;
    h = h == mx ? -INFINITY : h;
  }
  return th;
}

struct Cand {
  float v;
  int i;
};

// One 8-byte store that other XCDs' coherent loads see once it is acknowledged.
template <typename T>
__device__ __forceinline__ void store_pair(T* p, uint32_t lo, uint32_t hi) {
  static_assert(sizeof(T) == 8, "a pair");
  __hip_atomic_store(reinterpret_cast<unsigned long long*>(p), (static_cast<unsigned long long>(hi) << 32) | lo,
                     __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT);
}

// The k best of the n (<= kTreeCap) buffered candidates, by rank: each candidate
// counts the candidates better than it (indices are distinct, so ranks are too) and
// the ranks below k take their places; places past n get empty entries.  Ends with
// a barrier.
// The buffer is read two entries per 16-byte load and compared without branches, so
// the loads of an unrolled step are all in flight together.
__device__ __forceinline__ int better01(float av, int ai, float bv, int bi) {
  return static_cast<int>(av > bv) | (static_cast<int>(av == bv) & static_cast<int>(ai < bi));
}
__device__ __forceinline__ void rank_select(const Cand* buf, int n, int k, TreeShared& sh) {
  const int n2 = n & ~1;
  for (int c = threadIdx.x; c < n; c += kTreeThreads) {
    const Cand me = buf[c];
    int r = 0;
#pragma unroll 4
    for (int j = 0; j < n2; j += 2) {
      const float4 w = *reinterpret_cast<const float4*>(buf + j);
      r += better01(w.x, __float_as_int(w.y), me.v, me.i) + better01(w.z, __float_as_int(w.w), me.v, me.i);
    }
    if (n & 1) r += better01(buf[n - 1].v, buf[n - 1].i, me.v, me.i);
    if (r < k) {
      sh.win_v[r] = me.v;
      sh.win_i[r] = me.i;
    }
  }
  for (int t = threadIdx.x; t < k; t += kTreeThreads)
    if (t >= n) {
      sh.win_v[t] = -INFINITY;
      sh.win_i[t] = INT_MAX;
    }
  __syncthreads();
}

// The k best entries of the threads' lists into sh.win_v / sh.win_i, best first.
// A threshold that some wavefront's heads reach k times leaves few entries; those
// are ranked in LDS.  If more than kTreeCap remain (ties), k rounds of take_best.
// Called with every thread active; ends with a barrier.
template <int KMAX>
__device__ __forceinline__ void select_from_lists(TopList<KMAX>& top, TreeShared& sh, Cand* buf, int k) {
  const int lane = threadIdx.x % kWave, wave = threadIdx.x / kWave;
  const float th = wave_kth_head(top.v[0], k);
  if (lane == 0) sh.bv[0][wave] = th;
  if (threadIdx.x == 0) sh.n = 0;
  __syncthreads();
  float theta = sh.bv[0][0];
#pragma unroll
  for (int w = 1; w < kTreeWaves; ++w) theta = fmaxf(theta, sh.bv[0][w]);
  // the entries at or above theta are a prefix of each sorted list
  int cnt = 0;
#pragma unroll
  for (int j = 0; j < KMAX; ++j) cnt += top.i[j] != INT_MAX && top.v[j] >= theta ? 1 : 0;
  int off = 0;
  if (cnt) off = atomicAdd(&sh.n, cnt);
#pragma unroll
  for (int j = 0; j < KMAX; ++j)
    if (j < cnt && off + j < kTreeCap) buf[off + j] = Cand{top.v[j], top.i[j]};
  __syncthreads();
  const int n = sh.n;
  if (n <= kTreeCap) {
    rank_select(buf, n, k, sh);
    return;
  }
  for (int j = 0; j < k; ++j) {
    float val;
    int idx;
    take_best(top, sh, j, val, idx);
    if (threadIdx.x == 0) {
      sh.win_v[j] = val;
      sh.win_i[j] = idx;
    }
  }
  __syncthreads();
}

template <int KMAX>
__global__ __launch_bounds__(kTreeThreads) void k_tree_expand(TreeArgs a) {
  __shared__ TreeShared sh;
  __shared__ float lse_row[kTreeMaxRows];
  __shared__ float stat_lds[2 * kTreeMaxBlocks];
  __shared__ float par_lds[kTreeMaxRows];
  __shared__ __align__(16) Cand cbuf[kTreeCap];
  const int blk = blockIdx.x;
  const int row = blk / a.chunks, ch = blk % a.chunks;
  const int v0 = ch * a.chunk_len, v1 = min(a.V, v0 + a.chunk_len);

  // Phase 1: this workgroup's slice of row `row`.
  // kTreeLoads 16-byte loads per thread are in flight before any is used; loads
  // past the chunk read zeros (buffer resource ends at v1) and are skipped.
  const __amdgpu_buffer_rsrc_t lr = buffer_rsrc(a.logits + static_cast<size_t>(row) * a.V, v1 * 2);
  float m = -INFINITY, s = 0.f;
  TopList<KMAX> top;
  top.clear();
  // theta: a value that k of the logits seen by the wavefront reach (the lists keep
  // them), so nothing below it can be among the wavefront's k best.  It is set from
  // the k-th largest of the lanes' maxima of their first eight logits and raised once
  // per batch from the k-th largest of the lanes' list heads; the (divergent)
  // insertions of the logits at or above it stay rare.
  float theta = -INFINITY;
  // The trip count is the same for every lane (wave_max needs all lanes active);
  // each lane skips the logits past the chunk.
  for (int vb0 = v0; vb0 < v1; vb0 += kTreeThreads * 8 * kTreeLoads) {
    const int vb = vb0 + static_cast<int>(threadIdx.x) * 8;
    u32x4_t q[kTreeLoads];
#pragma unroll
    for (int u = 0; u < kTreeLoads; ++u)
      q[u] = __builtin_amdgcn_raw_buffer_load_b128(lr, static_cast<uint32_t>(vb + u * kTreeThreads * 8) * 2,
                                                   0, 0);
#pragma unroll
    for (int u = 0; u < kTreeLoads; ++u) {
      const int v = vb + u * kTreeThreads * 8;
      const bool live = v < v1;
      float z[8];
#pragma unroll
      for (int e = 0; e < 8; ++e) {
        const uint32_t w = q[u][e / 2];
        z[e] = __uint_as_float(e % 2 ? (w & 0xFFFF0000u) : (w << 16)) * a.inv_t;  // bf16 -> f32
      }
      float m8 = z[0];
#pragma unroll
      for (int e = 1; e < 8; ++e) m8 = fmaxf(m8, z[e]);
      if (theta == -INFINITY)  // wave-uniform: until a first bound is found
        theta = wave_kth_head(live ? m8 : -INFINITY, a.k);
      if (!live) continue;
      // online softmax over the eight: one rescale per load
      const float mn = fmaxf(m, m8);
      float add = 0.f;
#pragma unroll
      for (int e = 0; e < 8; ++e) add += __expf(z[e] - mn);
      s = (m == -INFINITY ? 0.f : s * __expf(m - mn)) + add;
      m = mn;
      // the rare logits at or above theta go through one insertion site
      unsigned hit = 0;
#pragma unroll
      for (int e = 0; e < 8; ++e) hit |= (z[e] >= theta ? 1u : 0u) << e;
      while (hit) {
        const int e = __builtin_ctz(hit);
        hit &= hit - 1;
        float ze = z[0];
#pragma unroll
        for (int f = 1; f < 8; ++f) ze = e == f ? z[f] : ze;
        if (better(ze, v + e, top.v[KMAX - 1], top.i[KMAX - 1])) top.insert(ze, v + e);
      }
    }
    theta = fmaxf(theta, wave_kth_head(top.v[0], a.k));
  }
  // (m, s) over the workgroup: lanes, then wavefronts, in a fixed order.
  {
    const float wm = wave_max(m);
    s = wave_sum(m == -INFINITY ? 0.f : s * __expf(m - wm));
    m = wm;
  }
  const int lane = threadIdx.x % kWave, wave = threadIdx.x / kWave;
  if (lane == 0) {
    sh.wm[wave] = m;
    sh.ws[wave] = s;
  }
  __syncthreads();
  float bm = sh.wm[0], bs = sh.ws[0];
#pragma unroll
  for (int w = 1; w < kTreeWaves; ++w) softmax_merge(bm, bs, sh.wm[w], sh.ws[w]);
  select_from_lists(top, sh, cbuf, a.k);
  if (static_cast<int>(threadIdx.x) < a.k) {
    store_pair(a.cand + static_cast<size_t>(blk) * a.k + threadIdx.x, __float_as_uint(sh.win_v[threadIdx.x]),
               static_cast<uint32_t>(sh.win_i[threadIdx.x]));
  }
  if (threadIdx.x == 0) store_pair(a.stat + blk, __float_as_uint(bm), __float_as_uint(bs));

  // Completion: every workgroup waits for its own stores, the last one goes on.
  __builtin_amdgcn_s_waitcnt(0x0F70);  // vmcnt(0)
  __syncthreads();
  if (threadIdx.x == 0)
    sh.last = __hip_atomic_fetch_add(a.cnt, 1u, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT) ==
              static_cast<unsigned>(gridDim.x - 1);
  __syncthreads();
  if (!sh.last) return;

  // Phase 2.  The workgroups' results are read with the coherent cache policy; each read
  // is a trip to the coherent level of the memory system, so a thread requests the
  // statistics and the whole list of its workgroup (and what is needed of the others where
  // there are more than 256) before anything waits.
  const int nblk = gridDim.x;
  const __amdgpu_buffer_rsrc_t rst = buffer_rsrc(a.stat, nblk * 8);
  const __amdgpu_buffer_rsrc_t rca = buffer_rsrc(a.cand, nblk * a.k * 8);
  // list entry j of workgroup b; past the end zeros, skipped when used
  auto load_cand = [&](int b, int j) __attribute__((always_inline)) {
    const auto v = __builtin_amdgcn_raw_buffer_load_b64(rca, static_cast<uint32_t>(b * a.k + j) * 8, 0, kTreeCoherent);
    return Cand{__uint_as_float(v[0]), static_cast<int>(v[1])};
  };
  // A thread's slots: workgroups thread, thread + 256, ...  The lists of the first kHeld are
  // held in registers; those of later ones (more than 256 or 512 workgroups) are read
  // where they are needed, in loops that are not unrolled: this code runs once per call,
  // so its size costs instruction fetches.
  constexpr int kHeld = KMAX == 8 ? 2 : 1;
  static_assert(kTreeMaxRows <= kTreeMaxBlocks, "one parent score per block slot");
  const __amdgpu_buffer_rsrc_t rp_ = buffer_rsrc(a.parent, a.R * 4);
  Cand list[kHeld][KMAX];
  float hv[kHeld], kv[kHeld];  // their first and k-th candidates
  auto load_stat = [&](int b) __attribute__((always_inline)) {
    const auto st = __builtin_amdgcn_raw_buffer_load_b64(rst, static_cast<uint32_t>(b) * 8, 0, kTreeCoherent);
    const float par = __uint_as_float(__builtin_amdgcn_raw_buffer_load_b32(rp_, static_cast<uint32_t>(b) * 4, 0, 0));
    return f32x4_t{__uint_as_float(st[0]), __uint_as_float(st[1]), par, 0.f};
  };
  auto keep_stat = [&](int b, const f32x4_t& st) __attribute__((always_inline)) {
    if (b < nblk) {
      stat_lds[2 * b] = st[0];
      stat_lds[2 * b + 1] = st[1];
    }
    if (b < a.R) par_lds[b] = st[2];
  };
  {
    f32x4_t st[kHeld];
#pragma unroll
    for (int h = 0; h < kHeld; ++h) {
      const int b = threadIdx.x + h * kTreeThreads;  // past the end zeros, skipped when used
#pragma unroll
      for (int j = 0; j < KMAX; ++j)
        if (j < a.k) list[h][j] = load_cand(b, j);
      st[h] = load_stat(b);
    }
#pragma unroll
    for (int h = 0; h < kHeld; ++h) {
      hv[h] = list[h][0].v;
#pragma unroll
      for (int j = 0; j < KMAX; ++j)
        if (j == a.k - 1) kv[h] = list[h][j].v;
      keep_stat(threadIdx.x + h * kTreeThreads, st[h]);
    }
#pragma unroll 1
    for (int b = threadIdx.x + kHeld * kTreeThreads; b < nblk; b += kTreeThreads) keep_stat(b, load_stat(b));
  }
  if (threadIdx.x == 0) sh.n = 0;
  __syncthreads();
  // The log-sum-exp of every row from its chunks' pairs: a group of G lanes per row
  // (G the power of two >= chunks, at most a wavefront), each lane over chunks
  // lane, lane + G, ..., then DPP reductions over a wavefront or a butterfly over a smaller
  // group.  Both merges of a butterfly pair give the same bits, so every lane ends with
  // the same pair.
  {
    int G = 1;
    while (G < a.chunks && G < kWave) G <<= 1;
    const int rows_per_pass = kTreeThreads / G;
    const int gl = threadIdx.x % G, gi = threadIdx.x / G;
    for (int r0 = 0; r0 < a.R; r0 += rows_per_pass) {  // the same trip count for all lanes
      const int r = r0 + gi;
      float rm = -INFINITY, rs = 0.f;
      if (r < a.R)
        for (int c = gl; c < a.chunks; c += G)
          softmax_merge(rm, rs, stat_lds[2 * (r * a.chunks + c)], stat_lds[2 * (r * a.chunks + c) + 1]);
      if (G == kWave) {
        const float wm = wave_max(rm);
        rs = wave_sum(rm == -INFINITY ? 0.f : rs * __expf(rm - wm));
        rm = wm;
      } else {
        for (int off = 1; off < G; off <<= 1) {
          const float om = __shfl_xor(rm, off), os = __shfl_xor(rs, off);
          softmax_merge(rm, rs, om, os);
        }
      }
      if (r < a.R && gl == 0) lse_row[r] = rm + __logf(rs);
    }
  }
  __syncthreads();
  // theta: a score that k candidates reach, so nothing below it can be among the k
  // best: the best score of any block's k-th candidate (that block alone has k
  // candidates at or above it: a score grows with z within a row, also in rounding),
  // or a value that k lanes' best block heads reach, whichever is larger.
  {
    float tb = -INFINITY, hb = -INFINITY;
    auto bound = [&](int b, float head, float kth) __attribute__((always_inline)) {
      if (b >= nblk) return;
      const int r = b / a.chunks;
      tb = fmaxf(tb, par_lds[r] + (kth - lse_row[r]));
      hb = fmaxf(hb, par_lds[r] + (head - lse_row[r]));
    };
#pragma unroll
    for (int h = 0; h < kHeld; ++h) bound(threadIdx.x + h * kTreeThreads, hv[h], kv[h]);
#pragma unroll 1
    for (int b = threadIdx.x + kHeld * kTreeThreads; b < nblk; b += kTreeThreads)
      bound(b, load_cand(b, 0).v, load_cand(b, a.k - 1).v);
    tb = fmaxf(wave_max(tb), wave_kth_head(hb, a.k));
    if (lane == 0) sh.wm[wave] = tb;
  }
  __syncthreads();
  float theta2 = sh.wm[0];
#pragma unroll
  for (int w = 1; w < kTreeWaves; ++w) theta2 = fmaxf(theta2, sh.wm[w]);
  // Every stored candidate becomes a score; those at or above theta are kept: a prefix of
  // each block's list, since its candidates come best first.
  auto score = [&](int r, const Cand& c) __attribute__((always_inline)) {
    // an empty slot of a short chunk scores below everything
    return c.i == INT_MAX ? Cand{-INFINITY, INT_MAX} : Cand{par_lds[r] + (c.v - lse_row[r]), r * a.V + c.i};
  };
  auto each = [&](auto&& take) __attribute__((always_inline)) {
#pragma unroll
    for (int h = 0; h < kHeld; ++h)
      if (static_cast<int>(threadIdx.x) + h * kTreeThreads < nblk)
        take((threadIdx.x + h * kTreeThreads) / a.chunks, list[h]);
#pragma unroll 1
    for (int b = threadIdx.x + kHeld * kTreeThreads; b < nblk; b += kTreeThreads) {
      Cand later[KMAX];
#pragma unroll
      for (int j = 0; j < KMAX; ++j)
        if (j < a.k) later[j] = load_cand(b, j);
      take(b / a.chunks, later);
    }
  };
  // Usually only a few candidates reach theta: they go to the LDS buffer and are
  // ranked there.
  each([&](int r, const Cand (&own)[KMAX]) __attribute__((always_inline)) {
    int cnt = 0;
#pragma unroll
    for (int j = 0; j < KMAX; ++j)
      if (j < a.k) cnt += own[j].i != INT_MAX && par_lds[r] + (own[j].v - lse_row[r]) >= theta2 ? 1 : 0;
    if (cnt) {
      const int off = atomicAdd(&sh.n, cnt);
#pragma unroll
      for (int j = 0; j < KMAX; ++j)
        if (j < cnt && off + j < kTreeCap) cbuf[off + j] = score(r, own[j]);
    }
  });
  __syncthreads();
  const int n = sh.n;
  if (n <= kTreeCap) {
    rank_select(cbuf, n, a.k, sh);
  } else {
    // More ties than the buffer holds: the same candidates again, through the
    // threads' lists and k rounds of take_best.
    top.clear();
    each([&](int r, const Cand (&own)[KMAX]) __attribute__((always_inline)) {
#pragma unroll
      for (int j = 0; j < KMAX; ++j)
        if (j < a.k) {
          const Cand c = score(r, own[j]);
          if (c.i != INT_MAX && c.v >= theta2) top.insert(c.v, c.i);
        }
    });
    for (int j = 0; j < a.k; ++j) {
      float val;
      int idx;
      take_best(top, sh, j, val, idx);
      if (threadIdx.x == 0) {
        sh.win_v[j] = val;
        sh.win_i[j] = idx;
      }
    }
    __syncthreads();
  }
  if (static_cast<int>(threadIdx.x) < a.k) {
    const int idx = sh.win_i[threadIdx.x];
    a.out_parent[threadIdx.x] = idx / a.V;
    a.out_token[threadIdx.x] = idx % a.V;
    a.out_score[threadIdx.x] = sh.win_v[threadIdx.x];
  }
  if (threadIdx.x == 0) __hip_atomic_store(a.cnt, 0u, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT);
}

}  // namespace

void tree_plan(int R, int V, int k, int* chunks, int* chunk_len) {
  // Workgroups in all, at least 2048 logits (one 16-byte load per thread) each:
  //  - up to 32 rows 256, one list per thread of the second phase (see the head of this
  //    file), while the slices stay short: with lists of 32 (k > 16) the insertions of a long
  //    slice cost more, and how many depends on the logits (eight sets each, k = 32: R = 24,
  //    V = 32000 37 to 64 us with 256 and 43 to 53 with 512; R = 32, V = 152064 90 and 62;
  //    R = 16 31 to 49 and the same, 152064 48 to 60 and 52 to 55), so there up to 16 rows;
  //  - up to 128 rows at most 512, two lists per thread, which are held in registers: the
  //    16 slices a row that 512 / 33 rounds up to leave a third list for 16 threads, read
  //    only when needed (R = 33, k = 6 26.2 us, with 15 slices 24.2; R = 63 30.9 and 26.8);
  //  - with more rows the number is rounded up (171 rows of 152064 in two workgroups each
  //    42.8 us at k = 6 against 46.9, 300 rows 57 against 71), except for lists of 32, of
  //    which a thread holds one (R = 300, k = 32 212 us and 188).
  const int total = R <= 16 || (R <= 32 && k <= 16) ? kTreeThreads : 2 * kTreeThreads;
  int c = R <= 128 || k > 16 ? total / R : (total + R - 1) / R;
  const int cmax = (V + 2047) / 2048;
  if (c > cmax) c = cmax;
  if (c < 1) c = 1;
  int len = (V + c - 1) / c;
  len = (len + 7) / 8 * 8;
  *chunk_len = len;
  *chunks = (V + len - 1) / len;
}

size_t tree_workspace_bytes(int R, int V, int k) {
  int chunks = 0, len = 0;
  tree_plan(R, V, k, &chunks, &len);
  const size_t blocks = static_cast<size_t>(R) * chunks;
  return kSplitCounterBytes + blocks * 2 * sizeof(float) + blocks * k * (sizeof(float) + sizeof(int));
}

hipError_t launch_tree_expand(const TreeArgs& a, hipStream_t st) {
  const dim3 grid(a.R * a.chunks), block(kTreeThreads);
  if (a.k <= 8)
    hipLaunchKernelGGL(k_tree_expand<8>, grid, block, 0, st, a);
  else if (a.k <= 16)
    hipLaunchKernelGGL(k_tree_expand<16>, grid, block, 0, st, a);
  else
    hipLaunchKernelGGL(k_tree_expand<32>, grid, block, 0, st, a);
  return hipGetLastError();
}

}  // namespace subspec
