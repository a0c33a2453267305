// The substitute-layer linear y = x * dequant(q, s, z)^T (SubSpec Sec. 4.1) for draft
// batches of 33 to 128 tree tokens (fewer on request), on 32x32x16 bf16 matrix cores (k_qmma).
//
// Roles of the operands: the activations are the A operand (32 rows of x per row
// block, read from LDS), the unpacked codes the B operand (32 columns per column
// block, straight from the weight stream), so a lane's accumulators all belong to one
// output column (lane % 32) and the per-column scale is one register.  A 32x32x16
// instruction keeps the matrix pipe busy for 32 cycles, long enough for about four
// VALU instructions of the same wavefront to issue in its shadow.
//
// Dequantization is folded into the accumulation as in the other kernels: inside a
// group the weight is affine in the code, so for every (row m, column n, group g)
//     sum_{k in g} x*W^ = s*( sum_{k in g} x*(128+q) ) - s*(128+z) * sum_{k in g} x.
// The first term: MFMAs on the exact bf16 values 128+q into a per-group accumulator,
// then tot += s * acc (one FMA per output per group).  The second term for a pair of
// groups at once: one fp32 32x32x2 MFMA with A = the two groups' sums of x and
// B = -s*(128+z) of the two groups (a rank-2 update of the 32x32 output block).
// The sums of x per (row, group): tiles of up to 64 rows take them from the x chunk in LDS
// (SumX), taller ones, which have no registers left for it, from a small kernel per call
// (k_xsum), copied into LDS beside the chunk.
//
// What bounds it: two wavefronts per SIMD must keep the matrix pipe busy through LDS
// reads, unpacking, scale FMAs, loads and the chunk barriers.  The loop is pipelined so
// that none of these leaves it idle for long: A fragments are read a step ahead, also
// across the barrier; a group's scale FMAs run between the next group's first MFMAs; and
// a chunk's loads are spread over its steps.  us per call, before (burst of loads and
// block of FMAs per chunk, the next chunk's first A read after the barrier, gathered x
// sums) and after, weights in the last-level cache in part (a stack that rotates them takes
// 75.8 at M = 128 3-bit): 55296x5120 M = 128 3-bit 89.0 / 68.5, 2-bit g64 93.3 / 75.8, 4-bit
// 99.5 / 71.4, M = 64 3-bit 47.9 / 43.3; 5120x27648 3-bit M = 128 58.8 / 51.8, M = 64
// 37.8 / 31.6; 37888x3584 4-bit M = 128 50.0 / 45.6, M = 64 34.5 / 29.5.
//
// No branch inside the loop: a branch, also one the compiler makes of a conditional read
// or store, splits the step and costs about 40 registers (spills).
//
// Weight fetch: a 32-column block is two 16-column tiles of the packed layout.  The
// B operand of step s (k = 16s ... 16s+15 of a 128-k block) holds, in lanes 0-31, k
// 16s..16s+7 of the block's 32 columns and in lanes 32-63 k 16s+8..16s+15; in tile
// terms lane l takes slice (l % 16) + 16*(2h + l/32) of tile 2cb + (l % 32)/16, with
// h = s % 2, and uses step j = s / 2 of that slice.  Each lane therefore loads two
// slices per block, and every load instruction reads two contiguous runs of 32 slices.
// Every load's per-chunk offset is a scalar (soffset): the lane part of each address
// is computed once.
#pragma once

#include "qlinear_device.h"

namespace subspec {

typedef __attribute__((__vector_size__(16 * sizeof(float)))) float f32x16_t;

namespace qmma {

typedef __attribute__((address_space(3))) void* LdsPtr;

// LDS of one workgroup: a ring of XB chunks of x per team, each [rows][16 pieces of
// 8 k] with the pieces of row r permuted by piece ^ (r & 15) (the copy-in writes a
// row's 16 pieces per 16 lanes and an A fragment reads one piece of 16 consecutive rows
// per 16 lanes, both conflict free).  The chunk buffers are separate LDS objects on
// purpose: the copy into one runs while another is read, and only distinct objects let
// the compiler see that those reads need not wait for the copy.

template <int BITS>
__device__ __forceinline__ Slice<BITS> load_slice_s(__amdgpu_buffer_rsrc_t r, uint32_t voff, uint32_t soff) {
  Slice<BITS> s;
  if constexpr (BITS == 4) {
    const auto v = __builtin_amdgcn_raw_buffer_load_b128(r, voff, soff, kStreamPolicy);
    s.w[0] = v[0]; s.w[1] = v[1]; s.w[2] = v[2]; s.w[3] = v[3];
  } else if constexpr (BITS == 2) {
    const auto v = __builtin_amdgcn_raw_buffer_load_b64(r, voff, soff, kStreamPolicy);
    s.w[0] = v[0]; s.w[1] = v[1];
  } else {
    const auto v = __builtin_amdgcn_raw_buffer_load_b96(r, voff, soff, kStreamPolicy);
    s.w[0] = v[0]; s.w[1] = v[1]; s.w[2] = v[2];
  }
  return s;
}

template <int BITS, int GROUP, int MB, int NB, int WAVES>
struct MmaBody {
  static constexpr int ROWS = 32 * MB;
  static constexpr int GPC = kTileK / GROUP;  // groups per 128-k chunk
  static constexpr int SPG = 8 / GPC;         // 16-k steps per group
  static constexpr int XCH = ROWS * 16;       // 16-byte pieces per chunk buffer
  static constexpr int DMA = ROWS / (4 * WAVES);  // x copy loads per wavefront per chunk
  static_assert(DMA * 4 * WAVES == ROWS, "each copy load fills four rows");
  static_assert(WAVES >= 4, "a lane's copies share their row % 16");
  // A fragments are read D steps ahead: a step is MB MFMAs of 32 cycles, an LDS read some
  // 130 cycles and more under load.  M = 128 q|k|v (7168x5120, 32-row tiles) 20.8 us with
  // D = 1.
  static constexpr int D = MB == 1 ? 4 : MB == 2 ? 2 : 1;

  // One ring slot: the chunk's two slices per column block and the fp16 scale and
  // zero-point of the lane's column for each of the chunk's groups.
  struct W {
    Slice<BITS> w[NB][2];
    uint16_t s[GPC][NB];  // raw fp16 bits, converted only when the group is applied
    uint16_t z[GPC][NB];
  };

  // Lane parts of every address, fixed for the whole launch.
  struct Lanes {
    uint32_t w[NB][2];     // slice byte offsets in block 0 of the column block's tiles
    uint32_t sz[NB];       // byte offset of the lane's column in a row of scales
    uint32_t x;            // byte offset of the lane's first copied piece in chunk 0
    uint32_t xs;           // byte offset of the lane's copied sum of x in chunk 0
    int a;                 // LDS piece index of the lane's first A fragment in row block 0
  };

  static __device__ __forceinline__ int slot(int row, int piece) { return row * 16 + (piece ^ (row & 15)); }

  // The loads of one chunk, in PIECES independent pieces that the main loop issues a few
  // per step: chunk kb's weights, scales and zero-points, and the chunk's copy of x.
  //
  // The copy (all ROWS rows; rows past M read zeros) goes straight from memory into an
  // LDS buffer: each load instruction fills 1 KB (four consecutive rows) with 16 bytes
  // per lane in lane order, so lane l writes position l % 16 of its row and fetches the
  // piece that the swizzle puts there.  Load j of wavefront w covers rows
  // 4w + 4*WAVES*j + (0..3): a lane keeps the same row % 16, hence the same swizzled
  // piece, in all of its loads.  The row part of the offset stays in the lane offset,
  // which the buffer's range check covers (rows past M read zeros); the chunk's
  // position in the row is the scalar offset.
  // Who sums x over the groups: 64-row tiles the workgroup itself (SumX; a pre-pass
  // kernel costs 5 us there), taller ones, which have no registers for it, a pre-pass
  // (k_xsum), whose sums are copied into LDS with the chunk ([group][row], 64 per
  // wavefront; wavefronts past the last 64 repeat them, and what the last 64 hold past the
  // chunk's sums is never read).
  static constexpr bool SUMS = MB <= 2;
  static constexpr int XSW = (GPC * ROWS + kWave - 1) / kWave;
  static constexpr int PIECES = 2 * NB + GPC + (SUMS ? 0 : 1) + DMA;
  static constexpr int VM = 2 * NB + 2 * GPC * NB + (SUMS ? 0 : 1) + DMA;  // vector memory operations of one chunk
  static __device__ __forceinline__ void stage(u32x4_t* xb, const QBuffers& bu, const Lanes& ln, int K, int kb,
                                               int wave, int j) {
    asm volatile("" : "+s"(K));  // recomputed at each copy: kept, the DMA offsets cost as many registers
    __builtin_amdgcn_raw_ptr_buffer_load_lds(bu.x, (LdsPtr)(xb + (4 * wave + 4 * WAVES * j) * 16), 16,
                                             ln.x + static_cast<uint32_t>(j) * (8 * WAVES) * K,
                                             static_cast<uint32_t>(kb) * (kTileK * 2), 0, 0);
  }
  // (P is a constant after inlining.)
  static __device__ __forceinline__ void load_piece(int P, W& r, u32x4_t* xb, float* xsb, const QBuffers& bu,
                                                    const Lanes& ln, const QArgs& a, int kb, int wave) {
    if (P < 2 * NB) {
      r.w[P / 2][P % 2] = load_slice_s<BITS>(bu.w, ln.w[P / 2][P % 2], static_cast<uint32_t>(kb) * (256 * BITS));
    } else if (P < 2 * NB + GPC) {
      const int gi = P - 2 * NB;
      const uint32_t soff = static_cast<uint32_t>(kb * GPC + gi) * a.N * 2;
#pragma unroll
      for (int nb = 0; nb < NB; ++nb) {
        r.s[gi][nb] = __builtin_amdgcn_raw_buffer_load_b16(bu.s, ln.sz[nb], soff, 0);
        r.z[gi][nb] = __builtin_amdgcn_raw_buffer_load_b16(bu.z, ln.sz[nb], soff, 0);
      }
    } else if (!SUMS && P == 2 * NB + GPC) {
      __builtin_amdgcn_raw_ptr_buffer_load_lds(bu.xs, (LdsPtr)(xsb + kWave * (wave % XSW)), 4,
                                               ln.xs + static_cast<uint32_t>(kb * GPC) * a.M * 4, 0, 0, 0);
    } else {
      stage(xb, bu, ln, a.K, kb, wave, P - (PIECES - DMA));
    }
  }

  // What a wavefront carries from one chunk to the next: the A fragments of the next
  // chunk's first D steps, and the last group's sums acc with its scale sv, which are
  // added to tot between the next group's first MFMAs (apply).
  struct Carry {
    bf16x8_t A[D][MB];
    f32x16_t acc[MB][NB];
    float sv[NB];
  };

  // Row 32 i + r32, piece 2 s + hi of a chunk buffer lives at 512 i + 16 r32 +
  // ((2 s + hi) ^ (r32 & 15)) = 512 i + (ln.a ^ 2 s).
  static __device__ __forceinline__ bf16x8_t read_a(const u32x4_t* X, const Lanes& ln, int lane, int i, int s) {
    return __builtin_bit_cast(bf16x8_t, X[512 * i + (ln.a ^ (2 * s))]);
  }

  static __device__ __forceinline__ void apply(const Carry& cy, f32x16_t (&tot)[MB][NB], int i) {
#pragma unroll
    for (int nb = 0; nb < NB; ++nb)
#pragma unroll
      for (int r = 0; r < 16; ++r) tot[i][nb][r] = __builtin_fmaf(cy.sv[nb], cy.acc[i][nb][r], tot[i][nb][r]);
  }

  // The eight 16-k steps of one chunk (x buffer X, ring slot wc).  A step reads the A
  // fragments of the step D ahead before its own MFMAs, so the LDS latency runs under
  // them; after step 7 - D every fragment of the chunk is in registers, the barrier runs
  // and the next chunk's first D steps (x buffer Xn) are read.  A group's first step adds
  // the group before it to tot (one row block's 16 FMAs before each MFMA that overwrites
  // those sums): the FMAs then run beside the matrix pipe and no group ends in a block of
  // them.  cneg[gi][nb] receives -s*(128+z) of the chunk's groups; hook(step) runs in
  // every step, issue(step) in the steps up to the barrier, zero_point after step ZS: the
  // offsets it needs are known, the chunk before's (SUMS) or this one's (after the last
  // group's first step).
  static constexpr int ZS = SUMS || GPC == 1 ? 1 : 5;
  template <typename F, typename I, typename Z, typename R>
  static __device__ __forceinline__ void compute(const W& wc, const u32x4_t* X, const u32x4_t* Xn, int lane,
                                                 const Lanes& ln, Carry& cy, f32x16_t (&tot)[MB][NB],
                                                 float (&cneg)[GPC][NB], F&& hook, I&& issue, Z&& zero_point,
                                                 R&& barrier) {
    const f32x16_t zero = {};
    bf16x8_t A[8][MB], An[D][MB];
#pragma unroll
    for (int d = 0; d < D; ++d)
#pragma unroll
      for (int i = 0; i < MB; ++i) A[d][i] = cy.A[d][i];
    static_for<8>([&](auto sc) __attribute__((always_inline)) {
      constexpr int S = decltype(sc)::value;  // 16-k step within the chunk
      constexpr int gi = S / SPG;
      constexpr bool FIRST = S % SPG == 0;
      if constexpr (S + D < 8) {
#pragma unroll
        for (int i = 0; i < MB; ++i) A[S + D][i] = read_a(X, ln, lane, i, S + D);
      }
      bf16x8_t B[NB];
#pragma unroll
      for (int nb = 0; nb < NB; ++nb) B[nb] = b_operand<BITS, S / 2>(wc.w[nb][S % 2]);
#pragma unroll
      for (int i = 0; i < MB; ++i) {
        if constexpr (FIRST) apply(cy, tot, i);
#pragma unroll
        for (int nb = 0; nb < NB; ++nb)
          cy.acc[i][nb] =
              __builtin_amdgcn_mfma_f32_32x32x16_bf16(A[S][i], B[nb], FIRST ? zero : cy.acc[i][nb], 0, 0, 0);
        if constexpr (FIRST) __builtin_amdgcn_sched_barrier(0);
      }
      issue(sc);
      hook(sc);
      if constexpr (FIRST) {
#pragma unroll
        for (int nb = 0; nb < NB; ++nb) {
          cy.sv[nb] = half_bits_to_float(wc.s[gi][nb]);
          const float z = half_bits_to_float(wc.z[gi][nb]);
          cneg[gi][nb] = -(cy.sv[nb] * (kCodeBias + z));
        }
      }
      // Keep each step's unpacking and reads next to its MFMAs: hoisting a whole chunk's
      // worth of them costs more registers than two wavefronts per SIMD leave.
      __builtin_amdgcn_sched_barrier(0);
      if constexpr (S == ZS) {
        zero_point();
        __builtin_amdgcn_sched_barrier(0);
      }
      if constexpr (S == 7 - D) {
        barrier();
#pragma unroll
        for (int d = 0; d < D; ++d)
#pragma unroll
          for (int i = 0; i < MB; ++i) An[d][i] = read_a(Xn, ln, lane, i, d);
      }
    });
#pragma unroll
    for (int d = 0; d < D; ++d)
#pragma unroll
      for (int i = 0; i < MB; ++i) cy.A[d][i] = An[d][i];
  }

  // The sums of x over each group of a chunk (x buffer X), [group][row]: LPR lanes a row,
  // 128 / LPR k each (bf16 dot products with ones, then lane exchanges within the row's
  // lanes of the group), the rows dealt to the team's wavefronts.  The lanes of 16
  // consecutive ones read 16 different pieces, so every read is free of bank conflicts.
  // Spread over the steps of the chunk, two pieces a step, summed one step after they are
  // read: done at once, the chain of reads and dot products stalls the wavefront (32B
  // gate|up at M = 128 75.5 us).
  struct SumX {
    static constexpr int LPR = ROWS >= 16 * WAVES ? 4 : 8;
    static constexpr int PPL = 16 / LPR;    // pieces of one lane and row
    static constexpr int RPW = kWave / LPR;  // rows of one wavefront at a time
    static constexpr int ROUNDS = ROWS / (RPW * WAVES);
    static_assert(!SUMS || (ROWS % (RPW * WAVES) == 0 && PPL % 2 == 0 && PPL * ROUNDS <= 10),
                  "whole rounds, within the steps");
    static constexpr int LPG = LPR / GPC;  // lanes of one group
    u32x4_t v[2];
    float sum[2];
    template <int S>
    __device__ __forceinline__ void step(const u32x4_t* X, float* xsum, int wave, int lane) {
      const int q = lane % LPR;
      if constexpr (S >= 2 && 2 * (S - 2) < PPL * ROUNDS) {
        constexpr int P = 2 * (S - 2), J = P / PPL;
        constexpr bool FIRST = P % PPL == 0;
#pragma unroll
        for (int t = 0; t < 2; ++t) sum[t] = piece_sum(v[t], FIRST ? 0.f : sum[t]);
        if constexpr (P % PPL == PPL - 2) {
          // the group's lanes all end with its sum and all store it: no branch
          xsum[q / LPG * ROWS + RPW * (wave + WAVES * J) + lane / LPR] = span_reduce<LPG>(sum[0] + sum[1]);
        }
      }
      if constexpr (S >= 1 && 2 * (S - 1) < PPL * ROUNDS) {
        constexpr int P = 2 * (S - 1), J = P / PPL;
#pragma unroll
        for (int t = 0; t < 2; ++t)
          v[t] = X[slot(RPW * (wave + WAVES * J) + lane / LPR, PPL * q + P % PPL + t)];
      }
    }
  };

  // Zero-point term of a pair of groups: lanes 0-31 carry the first group, lanes
  // 32-63 the second; xs[i] is the sum of x of the lane's row in block i and the
  // lane half's group, cop is -s*(128+z) of the lane half's group.  tot += X * C as
  // one fp32 32x32x2 MFMA per output block.
  static __device__ __forceinline__ void apply_pair(const float (&xs)[MB], const float (&cop)[NB],
                                                    f32x16_t (&tot)[MB][NB]) {
#pragma unroll
    for (int i = 0; i < MB; ++i)
#pragma unroll
      for (int nb = 0; nb < NB; ++nb)
        tot[i][nb] = __builtin_amdgcn_mfma_f32_32x32x2f32(xs[i], cop[nb], tot[i][nb], 0, 0, 0);
  }
};

// s_waitcnt immediate: at most `vm` vector memory operations outstanding, no LDS one.
constexpr int wait_vm_lds(int vm) { return (vm & 15) | (7 << 4) | ((vm >> 4) << 14); }

// Barrier between chunks.  Each wavefront first waits for its own copies into the buffer
// the next chunk uses and for its LDS reads.  Vector memory operations complete in issue
// order, so waiting until only the VM operations issued after those copies are
// outstanding is exact; a fenced __syncthreads() would drain all of them, and leaving the
// wait to the compiler (its own tracking of copies into LDS) missed copies whose
// instructions are spread over the steps.  (tests/test_compiled_waits.py counts the loads
// in the built library.)  The empty assembly statements keep the compiler from moving LDS
// accesses across the barrier.
template <int VM>
__device__ __forceinline__ void chunk_barrier() {
  static_assert(VM < 64, "vmcnt has six bits");
  asm volatile("" ::: "memory");
  __builtin_amdgcn_s_waitcnt(wait_vm_lds(VM));
  asm volatile("" ::: "memory");
  __builtin_amdgcn_s_barrier();
  asm volatile("" ::: "memory");
}

// XB: depth of the x ring and of each wavefront's weight ring, in 128-k chunks.  The
// barrier after chunk c waits for the copy of chunk c + 1, issued XB - 1 chunks
// earlier; the only weight load issued before that copy and not yet needed is the one
// for chunk c + 1 itself, so every weight load has XB - 1 chunks to arrive.
// WAVES: wavefronts per workgroup, one 32-column block each (NB = 1).  TEAMS = 1: all
// of them share the workgroup's x ring.  TEAMS > 1: teams of WAVES / TEAMS wavefronts on
// the same column blocks, each with an x ring of its own, take consecutive parts of the
// workgroup's k-blocks, and add their sums through LDS in team order at the end (more
// wavefronts per column group without more partial sums).
template <int BITS, int GROUP, int MB, int NB, int XB, int WAVES, int TEAMS>
// Four wavefronts: two workgroups per CU (two wavefronts per SIMD) fit the LDS of a
// two-chunk ring; a deeper ring takes one workgroup per CU and may use the SIMD's
// whole register file.  Eight wavefronts: one workgroup per CU, two per SIMD.
__global__ __launch_bounds__(WAVES * kWave)
__attribute__((amdgpu_waves_per_eu(WAVES == 8 || XB <= 2 ? 2 : 1))) void k_qmma(QArgs args) {
  const QArgs a = row_block(args);
  static_assert(XB % 2 == 0 && XB >= 2 && XB <= 6, "chunk parity (pairs of 128-k groups) follows the ring slot");
  static_assert(WAVES == 4 || WAVES == 8, "wavefronts per workgroup");
  static_assert(TEAMS == 1 || NB == 1, "teams of one column block per wavefront");
  constexpr int TW = WAVES / TEAMS;  // wavefronts per team (its column blocks)
  using Body = MmaBody<BITS, GROUP, MB, NB, TW>;
  constexpr int GPC = Body::GPC;
  constexpr bool SUMS = Body::SUMS;
  constexpr int XCH = Body::XCH;
  constexpr int PF = XB;
  constexpr int SPREAD = 8 - Body::D;  // steps of a chunk that issue loads: up to the barrier
  constexpr int NBUF = XB * TEAMS;  // LDS chunk buffers; team t uses [t * XB, t * XB + XB)
  static_assert(NBUF <= 8, "LDS chunk buffers");
  __shared__ u32x4_t xb0[XCH], xb1[XCH], xb2[NBUF > 2 ? XCH : 1], xb3[NBUF > 3 ? XCH : 1],
      xb4[NBUF > 4 ? XCH : 1], xb5[NBUF > 5 ? XCH : 1], xb6[NBUF > 6 ? XCH : 1], xb7[NBUF > 7 ? XCH : 1];
  constexpr int XSC = SUMS ? GPC * Body::ROWS : Body::XSW * kWave;  // sums of x of one chunk, [group][row]
  __shared__ float xs0[XSC], xs1[XSC], xs2[NBUF > 2 ? XSC : 1], xs3[NBUF > 3 ? XSC : 1], xs4[NBUF > 4 ? XSC : 1],
      xs5[NBUF > 5 ? XSC : 1], xs6[NBUF > 6 ? XSC : 1], xs7[NBUF > 7 ? XSC : 1];
  // Chunk buffer I, selected at compile time: separate LDS objects, so that the
  // compiler can tell the buffers' accesses apart.
  auto lds = [&](auto ic) __attribute__((always_inline)) -> u32x4_t* {
    constexpr int I = decltype(ic)::value;
    static_assert(I < NBUF, "chunk buffer index");
    if constexpr (I == 0) return xb0;
    else if constexpr (I == 1) return xb1;
    else if constexpr (I == 2) return xb2;
    else if constexpr (I == 3) return xb3;
    else if constexpr (I == 4) return xb4;
    else if constexpr (I == 5) return xb5;
    else if constexpr (I == 6) return xb6;
    else return xb7;
  };
  auto lds_xs = [&](auto ic) __attribute__((always_inline)) -> float* {
    constexpr int I = decltype(ic)::value;
    static_assert(I < NBUF, "chunk buffer index");
    if constexpr (I == 0) return xs0;
    else if constexpr (I == 1) return xs1;
    else if constexpr (I == 2) return xs2;
    else if constexpr (I == 3) return xs3;
    else if constexpr (I == 4) return xs4;
    else if constexpr (I == 5) return xs5;
    else if constexpr (I == 6) return xs6;
    else return xs7;
  };

  const int lane = threadIdx.x % kWave;
  const int wave = __builtin_amdgcn_readfirstlane(static_cast<int>(threadIdx.x / kWave));
  const int team = wave / TW, tw = wave % TW;
  const int r32 = lane & 31, hi = lane >> 5;
  const WorkItem wi(a);
  const int ng = wi.ng;
  // The team's k-blocks: a TEAMS-th of the workgroup's (rounded up) each, the last ones
  // the rest (possibly none).  All run team 0's number of chunk steps, so that their
  // barriers pair up; a team past its last chunk skips the arithmetic.
  const int nwg = wi.kb_end - wi.kb0;
  const int nsteps = (nwg + TEAMS - 1) / TEAMS;
  const int kb0 = wi.kb0 + team * nsteps;
  const int nchunks = min(max(nwg - team * nsteps, 0), nsteps);
  const int last = nchunks - 1;
  const QBuffers bu(a, BITS, GROUP);
  // Block of the team's chunk c, held inside the workgroup's range: loads past the
  // team's last chunk repeat it (L2 hits, never used).
  auto blk = [&](int c) __attribute__((always_inline)) {
    return min(kb0 + max(min(c, last), 0), wi.kb_end - 1);
  };

  // Column blocks of this wavefront: 32 columns each, tiles 2cb and 2cb + 1.  A
  // block past N (half of the last one when N % 32 == 16) reads a valid tile and is
  // never stored.
  typename Body::Lanes ln;
  bool ok[NB];
  int col[NB];
#pragma unroll
  for (int nb = 0; nb < NB; ++nb) {
    const int cb = (ng * TW + tw) * NB + nb;
    const int t = 2 * cb + (r32 >> 4);
    ok[nb] = t < a.n_tiles;
    const int tc = ok[nb] ? t : a.n_tiles - 1;
    col[nb] = tc * kTileN + (lane & 15);
    ln.sz[nb] = static_cast<uint32_t>(col[nb]) * 2;
#pragma unroll
    for (int h = 0; h < 2; ++h)
      ln.w[nb][h] = static_cast<uint32_t>(tc) * a.KB * (256 * BITS) + ((lane & 15) + 16 * (2 * h + hi)) * (4 * BITS);
  }
  {
    const int row = 4 * tw + (lane >> 4), pc = (lane & 15) ^ (row & 15);
    ln.x = (static_cast<uint32_t>(row) * a.K + pc * 8) * 2;
    ln.a = r32 * 16 + (hi ^ (r32 & 15));
    const int xi = kWave * (tw % Body::XSW) + lane;  // this lane's sum in the chunk's [group][row]
    ln.xs = (static_cast<uint32_t>(xi / Body::ROWS) * a.M + xi % Body::ROWS) * 4;
  }

  f32x16_t tot[MB][NB];
#pragma unroll
  for (int i = 0; i < MB; ++i)
#pragma unroll
    for (int nb = 0; nb < NB; ++nb) tot[i][nb] = f32x16_t{};

  // The main loop of team T (a compile-time constant, so that its ring buffers are
  // distinct LDS objects the compiler can tell apart).
  auto run = [&](auto tc) __attribute__((always_inline)) {
    constexpr int T = decltype(tc)::value;
    // ring slot I of team T: chunk c in slot c % XB
    auto ring = [&](auto ic) __attribute__((always_inline)) -> u32x4_t* {
      return lds(std::integral_constant<int, T * XB + decltype(ic)::value % XB>{});
    };
    auto ring_xs = [&](auto ic) __attribute__((always_inline)) -> float* {
      return lds_xs(std::integral_constant<int, T * XB + decltype(ic)::value % XB>{});
    };
    // Prologue: chunks 0 .. XB - 2 of x and of the weights in flight.  Unconditional
    // loads keep the compiler's count of outstanding loads exact.
    typename Body::W w[PF];
    static_for<XB - 1>([&](auto u) __attribute__((always_inline)) {
      constexpr int U = decltype(u)::value;
      static_for<Body::PIECES>([&](auto pc) __attribute__((always_inline)) {
        Body::load_piece(decltype(pc)::value, w[U], ring(u), ring_xs(u), bu, ln, a, blk(U), tw);
      });
    });
    if constexpr (SUMS)  // chunk 0's zero-point step reads the sums of "chunk -1"
      for (int i = lane; i < XSC; i += kWave) ring_xs(std::integral_constant<int, XB - 1>{})[i] = 0.f;
    chunk_barrier<(XB - 2) * Body::VM>();  // chunk 0 landed; chunks 1 .. XB - 2 in flight

    typename Body::Carry cy;
#pragma unroll
    for (int i = 0; i < MB; ++i) {
#pragma unroll
      for (int d = 0; d < Body::D; ++d)
        cy.A[d][i] = Body::read_a(ring(std::integral_constant<int, 0>{}), ln, lane, i, d);
#pragma unroll
      for (int nb = 0; nb < NB; ++nb) cy.acc[i][nb] = f32x16_t{};
    }
    // -s*(128+z) of the chunk before, and for 128-k groups that and the sums of x of the
    // first group of an open pair
    float cprev[GPC][NB], cfirst[NB], xfirst[MB];
#pragma unroll
    for (int nb = 0; nb < NB; ++nb) {
      cfirst[nb] = 0.f;
#pragma unroll
      for (int gi = 0; gi < GPC; ++gi) cprev[gi][nb] = 0.f;
    }
#pragma unroll
    for (int i = 0; i < MB; ++i) xfirst[i] = 0.f;
#pragma unroll
    for (int nb = 0; nb < NB; ++nb) cy.sv[nb] = 0.f;

    // One chunk cc (ring slot U = cc % XB, parity U).  Its steps issue the loads of chunk
    // cc + XB - 1 into the ring slots of chunk cc - 1, a few per step: as one burst after
    // the barrier they stall every wavefront of the CU on the address units at once.
    // Once every A fragment of the chunk is in registers the barrier waits for chunk
    // cc + 1 of x.  Once a pair of groups is complete its zero-point term is added.
    auto step = [&](auto u, int cc) __attribute__((always_inline)) {
      constexpr int U = decltype(u)::value;
      constexpr int V = (U + XB - 1) % XB;
      const int cn = cc + XB - 1;
      const int kbn = blk(cn);
      auto issue = [&](auto sc) __attribute__((always_inline)) {
        constexpr int S = decltype(sc)::value;
        static_for<Body::PIECES>([&](auto pc) __attribute__((always_inline)) {
          constexpr int P = decltype(pc)::value;
          if constexpr (P * SPREAD / Body::PIECES == S)
            Body::load_piece(P, w[V], ring(std::integral_constant<int, V>{}),
                             ring_xs(std::integral_constant<int, V>{}), bu, ln, a, kbn, tw);
        });
      };
      const bool active = TEAMS == 1 || cc < nchunks;
      auto barrier = [&]() __attribute__((always_inline)) {
        chunk_barrier<(XB - 2) * Body::VM>();  // in flight: chunks cc + 2 .. cc + XB - 1
      };
      if (active) {
        // Zero-point term: of this chunk (sums of x copied with it), or with SUMS of chunk
        // cc - 1, whose sums the barrier at its end made visible.
        constexpr int XU = SUMS ? (U + XB - 1) % XB : U;
        float cneg[GPC][NB], xs[MB];
        auto& cz = [&]() __attribute__((always_inline)) -> float(&)[GPC][NB] {
          if constexpr (SUMS) return cprev;
          else return cneg;
        }();
        const float* X = ring_xs(std::integral_constant<int, XU>{});
#pragma unroll
        for (int i = 0; i < MB; ++i) xs[i] = X[(GPC == 2 ? hi * Body::ROWS : 0) + 32 * i + r32];
        typename Body::SumX sx;
        Body::compute(w[U], ring(u), ring(std::integral_constant<int, (U + 1) % XB>{}), lane, ln, cy, tot, cneg, [&](auto sc) __attribute__((always_inline)) {
          constexpr int S = decltype(sc)::value;
          if constexpr (SUMS) sx.template step<S>(ring(u), ring_xs(u), tw, lane);
        }, issue, [&]() __attribute__((always_inline)) {
          float cop[NB];
          if constexpr (GPC == 2) {
#pragma unroll
            for (int nb = 0; nb < NB; ++nb) cop[nb] = hi ? cz[1][nb] : cz[0][nb];
            Body::apply_pair(xs, cop, tot);
          } else if constexpr (XU % 2 == 1) {
#pragma unroll
            for (int i = 0; i < MB; ++i) {
              asm volatile("" : "+v"(xs[i]));  // keeps the select from turning into a branch around the read
              xs[i] = hi ? xs[i] : xfirst[i];
            }
#pragma unroll
            for (int nb = 0; nb < NB; ++nb) cop[nb] = hi ? cz[0][nb] : cfirst[nb];
            Body::apply_pair(xs, cop, tot);
          } else {
#pragma unroll
            for (int i = 0; i < MB; ++i) xfirst[i] = xs[i];
#pragma unroll
            for (int nb = 0; nb < NB; ++nb) cfirst[nb] = cz[0][nb];
          }
        }, barrier);
#pragma unroll
        for (int gi = 0; gi < GPC; ++gi)
#pragma unroll
          for (int nb = 0; nb < NB; ++nb) cprev[gi][nb] = cneg[gi][nb];
      } else {
        static_for<SPREAD>(issue);
        barrier();
      }
    };
    for (int c = 0; c < nsteps; c += XB)
      static_for<XB>([&](auto u) __attribute__((always_inline)) {
        if (c + decltype(u)::value < nsteps) step(u, c + decltype(u)::value);
      });
    // the last group, and the zero-point term of the last chunk: with 128-k groups of the
    // open pair, or of its group alone when the number of chunks is odd
#pragma unroll
    for (int i = 0; i < MB; ++i) Body::apply(cy, tot, i);
    const bool alone = GPC == 1 && (nchunks & 1);
    if constexpr (SUMS) {
      if (nchunks > 0) {
        float cop[NB], xs[MB];
        static_for<XB>([&](auto u) __attribute__((always_inline)) {
          if (last % XB != decltype(u)::value) return;
#pragma unroll
          for (int i = 0; i < MB; ++i) xs[i] = ring_xs(u)[(GPC == 2 ? hi * Body::ROWS : 0) + 32 * i + r32];
        });
#pragma unroll
        for (int i = 0; i < MB; ++i) xs[i] = GPC == 2 || alone || hi ? xs[i] : xfirst[i];
#pragma unroll
        for (int nb = 0; nb < NB; ++nb)
          cop[nb] = GPC == 2 ? (hi ? cprev[GPC - 1][nb] : cprev[0][nb])
                    : alone  ? (hi ? 0.f : cprev[0][nb])
                             : (hi ? cprev[0][nb] : cfirst[nb]);
        Body::apply_pair(xs, cop, tot);
      }
    } else if (alone) {
      float cop[NB];
#pragma unroll
      for (int nb = 0; nb < NB; ++nb) cop[nb] = hi ? 0.f : cfirst[nb];
      Body::apply_pair(xfirst, cop, tot);
    }
  };
  if constexpr (TEAMS == 1) {
    run(std::integral_constant<int, 0>{});
  } else {
    static_for<TEAMS>([&](auto tc) __attribute__((always_inline)) {
      if (team == decltype(tc)::value) run(tc);
    });
  }
  if constexpr (TEAMS > 1) {
    // The other teams hand their sums to team 0 through the LDS of their rings, RPB of a
    // wavefront's 16 MB registers per chunk buffer.  Copies into the rings issued past the
    // last chunk may still be landing, so every wavefront first waits for its own.
    constexpr int RPB = XCH * 4 / (TW * kWave);
    static_assert(RPB * XB >= 16 * MB && RPB > 0, "a team's sums fit its ring");
    __builtin_amdgcn_s_waitcnt(kWaitVmcnt0);
    __syncthreads();
    static_for<TEAMS - 1>([&](auto uc) __attribute__((always_inline)) {
      constexpr int T = decltype(uc)::value + 1;
      if (team != T) return;
      static_for<16 * MB>([&](auto ec) __attribute__((always_inline)) {
        constexpr int E = decltype(ec)::value;
        float* red = reinterpret_cast<float*>(lds(std::integral_constant<int, T * XB + E / RPB>{}));
        red[(tw * RPB + E % RPB) * kWave + lane] = tot[E / 16][0][E % 16];
      });
    });
    __syncthreads();
    if (team == 0)
      static_for<TEAMS - 1>([&](auto uc) __attribute__((always_inline)) {
        constexpr int T = decltype(uc)::value + 1;
        static_for<16 * MB>([&](auto ec) __attribute__((always_inline)) {
          constexpr int E = decltype(ec)::value;
          const float* red = reinterpret_cast<const float*>(lds(std::integral_constant<int, T * XB + E / RPB>{}));
          tot[E / 16][0][E % 16] += red[(tw * RPB + E % RPB) * kWave + lane];
        });
      });
  }

  // D layout of the 32x32 MFMA: lane l holds column l % 32 and, in register r, row
  // 8 * (r / 4) + 4 * (l / 32) + r % 4 of the block.  The stores go through a buffer
  // resource over the output (bf16 y, or this split's fp32 partial sums) with the
  // whole offset in the vector offset, which the range check covers (the scalar
  // offset is not checked): rows at or past M fall outside the resource and are
  // dropped, and so are the lanes of a column block past N, given an offset outside
  // it.  All offsets stay below 2^31 (no wrap-around into the range) when the tile's
  // rows span less than 2 GiB; larger outputs take per-element stores.
  if (team == 0) {
    const bool split = wi.nsplit > 1;
    const uint32_t esz = split ? 4 : 2;
    const uint64_t out_bytes = static_cast<uint64_t>(a.M) * a.N * esz;
    if (static_cast<uint64_t>(32 * MB) * a.N * esz < (1ull << 31)) {
      const uint32_t rowb = static_cast<uint32_t>(a.N) * esz;
      const __amdgpu_buffer_rsrc_t out =
          split ? buffer_rsrc(a.ws + static_cast<size_t>(wi.split) * a.M * a.N, static_cast<uint32_t>(out_bytes))
                : buffer_rsrc(a.y, static_cast<uint32_t>(out_bytes));
      constexpr uint32_t kOutside = 0x80000000u;
      uint32_t voff[NB];
#pragma unroll
      for (int nb = 0; nb < NB; ++nb)
        voff[nb] = ok[nb] ? static_cast<uint32_t>(col[nb]) * esz + static_cast<uint32_t>(4 * hi) * rowb : kOutside;
      auto store_all = [&](auto splitc) __attribute__((always_inline)) {
        constexpr bool SPLIT = decltype(splitc)::value;
#pragma unroll
        for (int i = 0; i < MB; ++i)
#pragma unroll
          for (int nb = 0; nb < NB; ++nb)
#pragma unroll
            for (int r = 0; r < 16; ++r) {
              const uint32_t off = voff[nb] + static_cast<uint32_t>(32 * i + 8 * (r / 4) + (r % 4)) * rowb;
              const float v = tot[i][nb][r];  // a plain value: bit casts of a vector element misbehave
              if constexpr (SPLIT)
                __builtin_amdgcn_raw_buffer_store_b32(__float_as_uint(v), out, off, 0, kCachePolicyAgent);
              else
                __builtin_amdgcn_raw_buffer_store_b16(float_to_bf16_bits(v), out, off, 0, 0);
            }
      };
      if (split)
        store_all(std::true_type{});
      else
        store_all(std::false_type{});
    } else {
#pragma unroll
      for (int i = 0; i < MB; ++i)
#pragma unroll
        for (int nb = 0; nb < NB; ++nb)
#pragma unroll
          for (int r = 0; r < 16; ++r) {
            const int m = 32 * i + 8 * (r / 4) + 4 * hi + (r % 4);
            if (ok[nb] && m < a.M) store_out(a, wi, m, col[nb], tot[i][nb][r]);
          }
    }
  }
  if (wi.nsplit > 1) finish_splitk<WAVES * kWave>(a, ng, TW * NB * 32);
}

}  // namespace qmma

typedef void (*QmmaKernel)(QArgs);

struct MmaVariant {
  int mb, nb, pf, waves, teams, bits, group;  // pf: depth of the x and weight rings (k_qmma's XB)
  QmmaKernel fn;
};

// The instantiations of one bit width (kernels_qmma_b<bits>.hip).
const MmaVariant* qmma_variants_b2(int* n);
const MmaVariant* qmma_variants_b3(int* n);
const MmaVariant* qmma_variants_b4(int* n);

}  // namespace subspec
