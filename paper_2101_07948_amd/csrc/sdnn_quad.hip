// gfx950 row-quad kernel of the sparse-weight x dense-activation product (SparseDNN, arXiv
// 2101.07948, Sec. 3.2.2): the kernel that calls on a default plan run on.
//
//   * A consumer wavefront holds a program of 4, 8, 16 or 32 rows of W over a tile of 64
//     columns of C.  Its lanes form groups of 16 (programs of 4 and 8 rows) or 4 (16 and 32
//     rows), a group per row of a set; one step multiplies one entry of each group's row, so
//     one ds_read_b128 reads four or sixteen different B rows, and an entry's weight and LDS
//     address reach its group by a DPP broadcast (gen_quad_asm.py).  The accumulators are
//     plain registers: no VGPR index mode, no scalar weights.
//   * Against a wave per panel of rows and 256 columns (spmm_panel_kernel), a workgroup's
//     tile is a quarter as wide for the same outputs, so it stages a quarter of the bytes of
//     B per output, and the LDS ring holds 512 rows of B instead of 128.
//   * Rows of about equal length share a program, and a program has the height that makes it
//     about as long as the others of its packing, so the waves of a workgroup, which the ring
//     couples to within 512 rows of B, carry equal work.
//   * B is staged by four producer wavefronts with direct global->LDS DMA, four 256-byte rows
//     per instruction, through a ring of kQuadRing chunks of kQuadChunk rows; producers and
//     consumers synchronise through LDS words as in spmm_panel_kernel (chunks landed; lowest
//     chunk a consumer still reads), every wait bounded by a poll budget.
//   * Each row sums its entries in ascending column order with fused multiply-adds, as in
//     every kernel of the library, so C is the same bit for bit.
//
// What bounds it: no unit alone.  A quad-step (four entries x 64 columns) reads 1 KB of B, 4.05
// cycles of a CU's LDS, and its FMAs, address and weight ops take 16.4 cycles of a SIMD (a quarter
// of the CU) in groups of 4 lanes and 22.7 in groups of 16, so the groups of 4 are taken where a
// workgroup has rows enough to fill its waves with them.  On the 768 x 3072 layer at 90 %, N = 4096
// (97 k cycles) the steps are 66 % of the SIMDs' time and their reads 65 % of LDS's, fillers
// included, with no bank conflicts; waves wait 31 % of theirs, and each CU has one item, whose start
// and drain nothing overlaps.  Smaller calls wait more (768 x 768, N = 1024: 54 %).  Measured against
// the panel kernel: that layer 66.5 -> 46.8-48.8 us, 768 x 768 at 90 %, N = 1024 13.6 -> 8.3 us, 2048 x
// 2048 at 70 %, N = 512 55.9 -> 36.1 us, 3072 x 768 at 97 %, N = 16384 with GELU 124.1 -> 100.1 us.
#include <hip/hip_runtime.h>
#include <stdint.h>
#include <stdlib.h>
#include <string.h>
#include <unistd.h>

#include <algorithm>

#include "sdnn_device.h"
#include "sdnn_internal.h"

namespace sdnn {
namespace {

template <int N>
using group_acc_t = float __attribute__((ext_vector_type(N)));

struct QuadConsumer {
  const uint32_t* stream;  // the program's first block
  const uint32_t* descs;   // its descriptors
  uint32_t vlane;          // 16 * (lane % 16): the lane's byte offset in a staged B row
  uint32_t lane4;          // 4 * lane
  uint32_t prog_addr;      // LDS address of this consumer's progress word
  uint32_t ready_addr;     // LDS address of the ready words
  uint32_t overrun_addr;   // LDS address of the workgroup's overrun word
  uint32_t poll_budget;    // failed readiness checks the wave may still poll through (all items)
  uint32_t chunk_base;     // ring chunk number of the item's chunk 0
  uint32_t next_progress;  // progress word written when the program is done
};

#include "quad_asm_gen.h"
static_assert(kQuadAsmTailBlocks <= kQuadTailBlocks, "stream tail shorter than the prefetch");
static_assert(kQuadAsmUnits == kQuadUnits, "block layout mismatch");
static_assert(kQuadAsmLoShift == kQuadLoShift && kQuadAsmHiShift == kQuadHiShift &&
                  kQuadAsmCountMask == kQuadMaxBlocks,
              "descriptor fields mismatch");
static_assert(kQuadAsmPoison == kPoison, "poison mismatch");

constexpr uint32_t kProgressEnd = 0x7fffffffu;
constexpr int kPollBudgetQuad = 1 << 22;
// LDS: the ring, a row of zeros (read by the filler entries), the control words (ready[4] at
// +0, progress[16] at +64, the overrun word at +128), and the second row of zeros.
constexpr int kCtl = kQuadZeroRow + kQuadRowBytes;
constexpr int kLdsBytes = (kQuadZeroRow | kQuadFlip) + kQuadRowBytes;
static_assert(kCtl + 256 <= (kQuadZeroRow | kQuadFlip) && kLdsBytes <= 160 * 1024, "LDS layout");

struct QuadArgs {
  int32_t K, N, nchunks, nprogs;
  int32_t ring_chunks;  // chunk numbers an item takes up: nchunks, rounded up to half the ring
  int32_t n_rb, n_tiles, total_wg, per_xcd, epi, cached;
  uint32_t poll_budget;
  int32_t H, W, NB;  // image geometry of a 3x3 convolution (B is then the input X)
};

// ---- producers --------------------------------------------------------------------------
// (M0, the DMAs' LDS address, is not a register the compiler allocates; nothing else in these
// kernels uses it)

template <int BYTES>
__device__ __forceinline__ void dma_saddr(uint32_t lds, uint32_t voff, uint64_t base) {
  if constexpr (BYTES == 16)
    asm volatile("s_mov_b32 m0, %0\n\ts_nop 0\n\tglobal_load_lds_dwordx4 %1, %2"
                 :: "s"(lds), "v"(voff), "s"(base) : "memory");
  else
    asm volatile("s_mov_b32 m0, %0\n\ts_nop 0\n\tglobal_load_lds_dword %1, %2"
                 :: "s"(lds), "v"(voff), "s"(base) : "memory");
}
// The four 1 KB DMAs of a producer's rows of a full chunk under one M0: the instruction
// offset (13 bits, signed) moves the global and the LDS address alike, so DMA j carries
// offset 1024 j, and voff[j] = the lane's offset - 1024 j + 4096 from base - 4096.
__device__ __forceinline__ void dma_rows(uint32_t lds, const uint32_t (&v)[4], uint64_t base) {
  asm volatile("s_mov_b32 m0, %0\n\ts_nop 0\n\t"
               "global_load_lds_dwordx4 %1, %5\n\t"
               "global_load_lds_dwordx4 %2, %5 offset:1024\n\t"
               "global_load_lds_dwordx4 %3, %5 offset:2048\n\t"
               "global_load_lds_dwordx4 %4, %5 offset:3072"
               :: "s"(lds), "v"(v[0]), "v"(v[1]), "v"(v[2]), "v"(v[3]), "s"(base - 4096)
               : "memory");
}
__device__ __forceinline__ void dma_vaddr(uint32_t lds, uint64_t addr) {
  asm volatile("s_mov_b32 m0, %0\n\ts_nop 0\n\tglobal_load_lds_dwordx4 %1, off"
               :: "s"(lds), "v"(addr) : "memory");
}
__device__ __forceinline__ void lds_write(uint32_t addr, uint32_t v) {
  asm volatile("ds_write_b32 %0, %1" :: "v"(addr), "v"(v) : "memory");
}
// min of the 16 progress words (the slots of absent consumers hold kProgressEnd)
__device__ __forceinline__ uint32_t min_progress(uint32_t addr) {
  typedef uint32_t u4 __attribute__((ext_vector_type(4)));
  u4 a, b, c, d;
  asm volatile("ds_read_b128 %0, %4\n\tds_read_b128 %1, %4 offset:16\n\t"
               "ds_read_b128 %2, %4 offset:32\n\tds_read_b128 %3, %4 offset:48\n\t"
               "s_waitcnt lgkmcnt(0)"
               : "=&v"(a), "=&v"(b), "=&v"(c), "=&v"(d) : "v"(addr) : "memory");
  uint32_t m = kProgressEnd;
#pragma unroll
  for (int i = 0; i < 4; ++i) m = min(m, min(min(a[i], b[i]), min(c[i], d[i])));
  return __builtin_amdgcn_readfirstlane(m);
}
// What the padding of a convolution reads.
__device__ const float g_zeros[4] __attribute__((aligned(16))) = {0.0f, 0.0f, 0.0f, 0.0f};

// Lane state of the convolution's staging for one tile: the lane's four columns are four
// images of one pixel (y, x).
struct ConvLane {
  uint64_t base = 0;   // X + 4 n - (W + 1) * NB * 4: tap (0, 0) of channel 0
  uint32_t taps = 0;   // bit t: tap t = 3 ky + kx reads pixel (y + ky - 1, x + kx - 1) of the image
};
__device__ __forceinline__ ConvLane conv_lane(const QuadArgs& a, const float* X, int n0, int lane) {
  ConvLane c;
  const int n = n0 + 4 * (lane & 15);
  const int q = n / a.NB, y = q / a.W, x = q - y * a.W;
  c.base = (uint64_t)(uintptr_t)X + 4ull * (uint32_t)n - 4ull * (uint32_t)(a.W + 1) * (uint32_t)a.NB;
#pragma unroll
  for (int t = 0; t < 9; ++t)
    if ((unsigned)(y + t / 3 - 1) < (unsigned)a.H && (unsigned)(x + t % 3 - 1) < (unsigned)a.W)
      c.taps |= 1u << t;
  return c;
}
// Row k of the virtual B is input channel k / 9 shifted by tap k % 9.  The four rows of a DMA
// have their own channels and taps, so the lane address is computed per row quad (a dozen
// vector instructions); lanes whose pixel lies outside the image read zeros.  Against the
// panel kernel's staging, one masked DMA per virtual row with zero fills and filler loads
// (256 x 256 filters at 90 % on 14 x 14, 16 images): 60.3 -> 21.8 us.
__device__ __forceinline__ void stage_conv(const QuadArgs& a, const ConvLane& c, int n0, int r0,
                                           uint32_t lds, int lane) {
  if (n0 + 4 * (lane & 15) >= a.N) return;
  const uint32_t col = 4u * (uint32_t)a.NB, row = (uint32_t)a.W * col, plane = (uint32_t)a.H * row;
#pragma unroll 4
  for (int j = 0; j < kQuadChunk / 4; ++j) {
    const uint32_t k = (uint32_t)min(r0 + 4 * j + (lane >> 4), a.K - 1);
    const uint32_t ic = k / 9u, t = k - 9u * ic, ky = (t * 11u) >> 5, kx = t - 3u * ky;
    const uint64_t at = c.base + (uint64_t)ic * plane + (ky * row + kx * col);
    dma_vaddr(lds + 1024u * j, (c.taps >> t) & 1u ? at : (uint64_t)(uintptr_t)g_zeros);
  }
}

// Stages rows [r0, r0 + kQuadChunk) of the tile at columns n0.. into the ring slot at LDS
// address `lds`: 16-byte pieces, four rows per DMA (lane group r: row r), or 4-byte pieces, a
// row per DMA.  Rows past K stage row K-1 again (no entry reads them); lanes past N stay out.
// Always kLoads<STAGE> DMAs.
template <int STAGE>
constexpr int kLoads = STAGE == kQuadDword ? kQuadChunk : kQuadChunk / 4;

template <int STAGE>
__device__ __forceinline__ void stage_chunk(const QuadArgs& a, const float* B, int n0, int r0,
                                            uint32_t lds, const uint32_t (&voff)[4], int lane) {
  const uint32_t row_bytes = (uint32_t)a.N * 4u;
  const uint64_t tile = (uint64_t)(uintptr_t)(B + n0);
  const uint32_t lrow = (uint32_t)lane >> 4, lcol = (uint32_t)(lane & 15) * 16u;
  if constexpr (STAGE == kQuadVec) {
    if (n0 + 4 * (lane & 15) < a.N) {
      if (r0 + kQuadChunk <= a.K) {
        uint64_t base = tile + (uint64_t)(uint32_t)r0 * row_bytes;
#pragma unroll
        for (int j = 0; j < kQuadChunk / 16; ++j, base += 16ull * row_bytes)
          dma_rows(lds + 4096u * j, voff, base);
      } else {
#pragma unroll
        for (int j = 0; j < kQuadChunk / 4; ++j) {
          const uint32_t row = (uint32_t)min(r0 + 4 * j + (int)lrow, a.K - 1);
          dma_vaddr(lds + 1024u * j, tile + (uint64_t)row * row_bytes + lcol);
        }
      }
    }
  } else {
    if (n0 + lane < a.N) {
#pragma unroll 8
      for (int j = 0; j < kQuadChunk; ++j) {
        const uint32_t row = (uint32_t)min(r0 + j, a.K - 1);
        dma_saddr<4>(lds + (uint32_t)j * kQuadRowBytes, 4u * (uint32_t)lane,
                     tile + (uint64_t)row * row_bytes);
      }
    }
  }
}

// Producer `prod` stages every kQuadProducers-th chunk, whole: chunk g goes to ring slot
// g % kQuadRing once g < min(progress) + kQuadRing.  (A chunk split between the producers
// would cost each of them the loop's 700 cycles of scalar work per chunk; so, that cost is
// paid once per kQuadProducers chunks.)  Its ready word is the next chunk it has not landed,
// so every chunk below the smallest ready word has landed.  Two chunks are in flight: a
// chunk's DMAs go out before the previous one's are waited for.  An item takes ring_chunks
// chunk numbers; those past nchunks hold no rows (an item's chunk c keeps ring slot
// c % kQuadRing, or c + 4).
template <int STAGE>
__device__ __forceinline__ void produce(const float* B, const QuadArgs& a, int prod, int lane, int item,
                        int nitems) {
  constexpr int L = kLoads<STAGE>;
  static_assert(L <= 32 || STAGE == kQuadDword, "vmcnt field");
  const uint32_t ready = kCtl + 4u * prod, prog0 = kCtl + 64, overrun = kCtl + 128;
  const uint32_t row_bytes = (uint32_t)a.N * 4u;
  const uint32_t total = (uint32_t)nitems * (uint32_t)a.ring_chunks;
  uint32_t limit = kQuadRing, budget = a.poll_budget;
  bool pending = false;  // the previous chunk has DMAs in flight
  int ci = prod;         // chunk within the item
  int n0 = item / a.n_rb * kQuadTileCols;
  ConvLane conv;
  if constexpr (STAGE == kQuadConv) conv = conv_lane(a, B, n0, lane);
  uint32_t voff[4];
#pragma unroll
  for (int j = 0; j < 4; ++j)
    voff[j] = (uint32_t)(lane & 15) * 16u + (((uint32_t)lane >> 4) + 4u * j) * row_bytes - 1024u * j + 4096u;
  for (uint32_t g = (uint32_t)prod; g < total; g += kQuadProducers) {
    if (g >= limit) {
      limit = min_progress(prog0) + kQuadRing;
      if (g >= limit) {
        if (pending) {  // nothing to stage: land the previous chunk
          asm volatile("s_waitcnt vmcnt(0)" ::: "memory");
          if (lane == 0) lds_write(ready, g);
          pending = false;
        }
        while ((limit = min_progress(prog0) + kQuadRing) <= g) {
          if (budget == 0) {
            // budget spent: stage anyway, after saying that a slot still being read may go
            lds_write(overrun, 1u);
            asm volatile("s_waitcnt lgkmcnt(0)" ::: "memory");
            break;
          }
          --budget;
          __builtin_amdgcn_s_sleep(1);
        }
      }
    }
    const bool real = ci < a.nchunks;
    const uint32_t slot = quad_slot(g % kQuadRing);
    if constexpr (STAGE == kQuadConv) {
      if (real) stage_conv(a, conv, n0, ci * kQuadChunk, slot, lane);
    } else {
      if (real) stage_chunk<STAGE>(a, B, n0, ci * kQuadChunk, slot, voff, lane);
    }
    if (pending) {  // the previous chunk has landed once at most this one's DMAs are left
      if (real) asm volatile("s_waitcnt vmcnt(%0)" :: "n"(L <= 63 ? L : 0) : "memory");
      else asm volatile("s_waitcnt vmcnt(0)" ::: "memory");
      if (lane == 0) lds_write(ready, g);
      pending = false;
    }
    if (real && STAGE != kQuadDword) {
      pending = true;
    } else {  // no rows, or 64 DMAs (the counter's range): land at once
      asm volatile("s_waitcnt vmcnt(0)" ::: "memory");
      if (lane == 0) lds_write(ready, g + kQuadProducers);
    }
    ci += kQuadProducers;
    if (ci >= a.ring_chunks) {  // the next item
      ci -= a.ring_chunks;
      item += a.total_wg;
      n0 = item / a.n_rb * kQuadTileCols;
      if constexpr (STAGE == kQuadConv) conv = conv_lane(a, B, n0, lane);
    }
  }
  asm volatile("s_waitcnt vmcnt(0)" ::: "memory");
  if (lane == 0) lds_write(ready, kProgressEnd);
  asm volatile("s_waitcnt lgkmcnt(0)" ::: "memory");
}

// ---- kernel -----------------------------------------------------------------------------

// The epilogue of a program's 4 NS rows, one copy per activation: with the activation chosen per
// element, each element was a basic block of its own, whose reciprocal and exponential nothing
// overlapped.  Lane group g of set q holds row q * kRows + g, the lane kVecs times four
// columns (of groups of 4 lanes, the i-th vector is quarter i ^ (g % 4)).
template <typename V, bool CACHED>
__device__ __forceinline__ void store_vec(float* c, float x, float y, float z, float w) {
  const nt_float4 v = {x, y, z, w};
  if constexpr (CACHED) *reinterpret_cast<V*>(c) = v;
  else __builtin_nontemporal_store(v, reinterpret_cast<V*>(c));
}
// (a 16-byte store needs 4-byte alignment only)
typedef nt_float4 __attribute__((aligned(4))) dword_float4;

template <int NS, int STAGE, int EPI, bool CACHED, int SETS, int ACCS>
__device__ __forceinline__ void store_program(const group_acc_t<ACCS> (&acc)[SETS], const int (&out)[SETS],
                                              const float (&bb)[SETS], float* C, int n0, int lane, int N) {
  constexpr int kGroup = NS <= 2 ? 16 : 4, kVecs = ACCS / 4;
  const int quarter = lane / kGroup % 4;
#pragma unroll
  for (int q = 0; q < SETS; ++q) {
    float v[ACCS];
#pragma unroll
    for (int k = 0; k < ACCS; ++k) v[k] = activation(acc[q][k] + bb[q], EPI);
    if (out[q] < 0) continue;
    float* c = C + (size_t)out[q] * N;
#pragma unroll
    for (int i = 0; i < kVecs; ++i) {
      const int n = n0 + 4 * (lane % kGroup) + 4 * kGroup * (kVecs > 1 ? i ^ quarter : 0);
      const float *e = v + 4 * i;
      if constexpr (STAGE == kQuadDword) {
        if (n + 4 <= N) {
          store_vec<dword_float4, CACHED>(c + n, e[0], e[1], e[2], e[3]);
        } else {
#pragma unroll
          for (int k = 0; k < 3; ++k)
            if (n + k < N) c[n + k] = e[k];
        }
      } else if (n < N) {
        store_vec<nt_float4, CACHED>(c + n, e[0], e[1], e[2], e[3]);
      }
    }
  }
}

template <int NS, int STAGE, bool CACHED, int SETS, int ACCS>
__device__ __forceinline__ void finish_program(const group_acc_t<ACCS> (&acc)[SETS], const int (&out)[SETS],
                                               const float (&bb)[SETS], float* C, int n0, int lane,
                                               const QuadArgs& a) {
  const int epi = epilogue_of(acc[0][0], a.epi);
  if (epi == SDNN_EPI_GELU)
    store_program<NS, STAGE, SDNN_EPI_GELU, CACHED>(acc, out, bb, C, n0, lane, a.N);
  else if (epi == SDNN_EPI_RELU)
    store_program<NS, STAGE, SDNN_EPI_RELU, CACHED>(acc, out, bb, C, n0, lane, a.N);
  else
    store_program<NS, STAGE, SDNN_EPI_NONE, CACHED>(acc, out, bb, C, n0, lane, a.N);
}

// A wave's place in its workgroup's items.
struct QuadCursor {
  int it, nitems, item, tile, prog, stratum;
  __device__ __forceinline__ void find(const QuadArgs& a) {  // the program of `item`
    tile = item / a.n_rb;
    const int rb = item - tile * a.n_rb;
    prog = stratum * a.n_rb + ((stratum & 1) ? a.n_rb - 1 - rb : rb);  // quad_program
  }
  __device__ __forceinline__ bool next(const QuadArgs& a) {
    item += a.total_wg;
    return ++it < nitems;
  }
};

// One program of a consumer wave over the items that run it in a row (when the row-blocks
// divide the workgroups, all of the wave's): its loop and the epilogue of its rows per item.
// The rows' tables are read once; read per item, their two dependent loads stood between the
// items of every wave.
template <int CAP, int NS, int STAGE>
__device__ __forceinline__ void run_program(QuadConsumer& ca, bool entries, const int32_t* rows,
                                            const int32_t* outs, float* C, const float* bias,
                                            QuadCursor& cur, int lane, const QuadArgs& a) {
  constexpr int kGroup = NS <= 2 ? 16 : 4, kRows = 64 / kGroup, kSets = 4 * NS / kRows;
  constexpr int kAccs = kQuadTileCols / kGroup;
  int out[kSets];
  float bb[kSets];
#pragma unroll
  for (int q = 0; q < kSets; ++q) {
    const int j = q * kRows + lane / kGroup;
    out[q] = outs[j];
    const int src = rows[j];
    bb[q] = bias && src >= 0 ? bias[src] : 0.0f;
  }
  const uint32_t vlane = (uint32_t)(lane % kGroup) * 16u + (kAccs > 4 ? (uint32_t)(lane / kGroup % 4) * 64u : 0u);
  const int prog = cur.prog;
  do {
    ca.chunk_base = (uint32_t)(cur.it * a.ring_chunks);
    ca.vlane = vlane ^ (ca.chunk_base & 4u ? kQuadFlip : 0u);
    ca.next_progress = cur.it + 1 < cur.nitems ? (uint32_t)((cur.it + 1) * a.ring_chunks) : kProgressEnd;
    group_acc_t<kAccs> acc[kSets];
#pragma unroll
    for (int q = 0; q < kSets; ++q)
#pragma unroll
      for (int k = 0; k < kAccs; ++k) acc[q][k] = 0.0f;
    if (entries) {
      if constexpr (NS == 1) consume_quads1(acc, ca);
      if constexpr (NS == 2) consume_quads2(acc, ca);
      if constexpr (NS == 4) consume_quads4(acc, ca);
      if constexpr (NS == 8) consume_quads8(acc, ca);
      // (between the loops the budget is in a VGPR: SGPRs are short and spill; but for the packing
      // of 32-row programs, whose VGPRs are)
      if constexpr (CAP == 8) ca.poll_budget = __builtin_amdgcn_readfirstlane(ca.poll_budget);
    } else if (lane == 0) {
      lds_write(ca.prog_addr, ca.next_progress);  // no entries: only epi(bias)
    }
    const int n0 = cur.tile * kQuadTileCols;
    if (a.cached)
      finish_program<NS, STAGE, true>(acc, out, bb, C, n0, lane, a);
    else
      finish_program<NS, STAGE, false>(acc, out, bb, C, n0, lane, a);
    if (!cur.next(a)) return;
    cur.find(a);
  } while (cur.prog == prog);
}

// STAGE: 16-byte staging and stores (N % 4 == 0, B and C 16-byte aligned) or 4-byte ones;
// CAP: the packing's largest programs, in quads.  blockDim.x = 64 * (consumers +
// kQuadProducers).  A workgroup takes the items (tile, row-block) numbered w, w + total_wg, ...
// in tile-major order; the consecutive workgroups of one XCD work on consecutive items and
// share their tiles' B rows in its L2.  Consumer w of a row-block takes the programs of one
// stratum of the list sorted by length, in snake order over the row-blocks, so that
// row-blocks carry equal work, and the strata go to the SIMDs (wave w runs on SIMD w % 4)
// in snake order too.
template <int CAP, int STAGE>
__global__ __launch_bounds__(1024) void spmm_quad_kernel(
    const uint32_t* __restrict__ stream, const uint32_t* __restrict__ descs,
    const QuadProgram* __restrict__ progs, const int32_t* __restrict__ rows,
    const int32_t* __restrict__ outs, const float* __restrict__ B, float* __restrict__ C,
    const float* __restrict__ bias, QuadArgs a) {
  // the loops form LDS addresses from the stream alone: the ring starts at LDS 0, which
  // holds because this is the kernel's only LDS object
  __shared__ __attribute__((aligned(16))) uint32_t lds[kLdsBytes / 4];
  const int bid = blockIdx.x;
  const int lin = (bid & 7) * a.per_xcd + (bid >> 3);
  if (lin >= a.total_wg) return;  // whole workgroup leaves before the barrier
  const int nc = (int)(blockDim.x >> 6) - kQuadProducers;
  const int wave = __builtin_amdgcn_readfirstlane(threadIdx.x >> 6);
  const int lane = threadIdx.x & 63;
  const int prod = wave - nc;
  const int items = a.n_tiles * a.n_rb;
  const int nitems = (items - lin + a.total_wg - 1) / a.total_wg;

  // LDS is read and written by assembly alone, at addresses from 0 up; handing the object's
  // address to an asm statement keeps it (and its size) in the kernel
  const uint32_t lds_base = (uint32_t)(uintptr_t)((__attribute__((address_space(3))) uint32_t*)lds);
  asm volatile("" ::"v"(lds_base) : "memory");
  const uint32_t progress = kCtl + 64u + 4u * (uint32_t)wave;
  if (prod >= 0) {
    if (lane == 0) lds_write(kCtl + 4u * prod, (uint32_t)prod);                    // nothing landed
    if (prod == 0 && lane >= nc && lane < 16) lds_write(kCtl + 64u + 4u * lane, kProgressEnd);  // absent
    if (prod == 0 && lane == 0) lds_write(kCtl + 128u, 0u);                        // no overrun
    if (prod == 1) lds_write(kQuadZeroRow + 4u * lane, 0u);                        // the rows of zeros
    if (prod == 2) lds_write((kQuadZeroRow | kQuadFlip) + 4u * lane, 0u);
  } else if (lane == 0) {
    lds_write(progress, 0u);
  }
  asm volatile("s_waitcnt lgkmcnt(0)" ::: "memory");
  __syncthreads();

  if (prod >= 0) {
    produce<STAGE>(B, a, prod, lane, lin, nitems);
    return;
  }

  const int g4 = wave >> 2, i4 = wave & 3;
  QuadCursor cur;
  cur.it = 0;
  cur.nitems = nitems;
  cur.item = lin;
  cur.stratum = (g4 & 1) && 4 * g4 + 4 <= nc ? 4 * g4 + 3 - i4 : wave;
  cur.find(a);
  uint32_t budget = a.poll_budget;
  while (cur.it < nitems) {
    if (cur.prog >= a.nprogs) {  // no program in this row-block
      if (lane == 0)
        lds_write(progress, cur.it + 1 < nitems ? (uint32_t)((cur.it + 1) * a.ring_chunks) : kProgressEnd);
      cur.next(a);
      cur.find(a);
      continue;
    }
    const QuadProgram P = progs[cur.prog];
    QuadConsumer ca;
    ca.stream = stream + (size_t)P.start * 64;
    ca.descs = descs + P.desc;
    ca.lane4 = (uint32_t)lane * 4u;
    ca.prog_addr = progress;
    ca.ready_addr = kCtl;
    ca.overrun_addr = kCtl + 128u;
    ca.poll_budget = budget;
    const int32_t* r = rows + (size_t)cur.prog * (4 * CAP);
    const int32_t* o = outs + (size_t)cur.prog * (4 * CAP);
    if (CAP == 8 && P.NS == 8) run_program<CAP, 8, STAGE>(ca, P.start >= 0, r, o, C, bias, cur, lane, a);
    else if (CAP >= 4 && P.NS == 4) run_program<CAP, 4, STAGE>(ca, P.start >= 0, r, o, C, bias, cur, lane, a);
    else if (CAP >= 2 && P.NS == 2) run_program<CAP, 2, STAGE>(ca, P.start >= 0, r, o, C, bias, cur, lane, a);
    else run_program<CAP, 1, STAGE>(ca, P.start >= 0, r, o, C, bias, cur, lane, a);
    budget = ca.poll_budget;
  }
}

template <int CAP, int STAGE>
hipError_t launch_cap(const DevQuads& d, const float* B, float* C, const float* bias,
                      const QuadArgs& args, int waves, int grid, hipStream_t stream) {
  hipLaunchKernelGGL((spmm_quad_kernel<CAP, STAGE>), dim3(grid), dim3(64 * (waves + kQuadProducers)),
                     0, stream, d.stream, d.descs, d.progs, d.rows, d.outs, B, C, bias, args);
  return hipGetLastError();
}

template <int STAGE>
hipError_t launch_stage(const DevQuads& d, const float* B, float* C, const float* bias,
                        const QuadArgs& args, int waves, int grid, hipStream_t stream) {
  switch (d.cap) {
    case 1: return launch_cap<1, STAGE>(d, B, C, bias, args, waves, grid, stream);
    case 2: return launch_cap<2, STAGE>(d, B, C, bias, args, waves, grid, stream);
    case 4: return launch_cap<4, STAGE>(d, B, C, bias, args, waves, grid, stream);
    case 8: return launch_cap<8, STAGE>(d, B, C, bias, args, waves, grid, stream);
  }
  return hipErrorInvalidValue;
}

// Whether C is stored through the caches or streamed past them.  The groups of 4 lanes store 64
// bytes of a row at a time.  Where rows of C do not begin at 64 bytes, those stores reach memory
// as parts of lines unless L2 joins them first (3000 x 128 at 90 %, N = 3092: 29.6 us streamed,
// 19.2 cached; N = 4095: 44.7 and 23.6; below 8 MB streaming is as fast or faster: 500 x 32,
// N = 1000: 5.6 and 5.9).  Aligned ones are streamed (with three sets of B and C in turn, which
// the 256 MB memory-side cache does not hold: 3072 x 768 at 97 %, N = 16384 96 us streamed, 123
// cached; 768 x 768 32 and 39; 3000 x 96 49 and 57; a small C is written back when the kernel
// ends: 256 x 256 9.3 and 10.4), but for a K so small that the store is all there is to do
// (3000 x 32 at 90 %, N = 16384: 54 and 49).  With still more buffers in turn, over 1 GiB, the half
// lines cost what the step gains: that layer 151 us streamed, 128 cached, 123 on the panel kernel; 768 x
// 768 36, 34 and 33.  (Two groups exchanging vectors, to store 128 bytes of a row at once: 125 us so,
// but 110 instead of 100 with three sets.)
bool cached_stores(const sdnn_plan_s* p, const float* C, int32_t N) {
  const int64_t bytes = (int64_t)p->M * N * 4;
  if (N % 16 != 0 || ((uintptr_t)C & 63) != 0) return bytes >= (int64_t)8 << 20;
  return p->K <= 32 && bytes >= (int64_t)48 << 20;
}

int env_or(const char* name, int dflt) {
  const char* s = getenv(name);
  return s ? atoi(s) : dflt;
}

// The packing and the consumer waves of a call: those that a cost model gives the least
// time.  In microseconds, for a workgroup's item (all measured on MI355X):
//     lat * chain + thr * mean program * max(waves / 4, 1)   blocks of 8 quad-steps
//   + sync * chunks + stage * ring chunks                    handshakes, staging
//   + store * rows + item                                    epilogue, start
// times the rounds of items over the CUs, + 3.5 for the launch.  lat, thr, sync, item: 0.080, 0.039,
// 0.082, 0.21 for programs of 4 and 8 rows, 0.112, 0.016, 0.074, 0.17 (0.58) for those of 16 (32);
// stage: 0.13, 4-byte pieces 0.29, a convolution 0.20; store: 0.0071 (32 rows 0.0054), a third more
// through the caches.  Fitted to 12900 timings over 440 problems (M = 16 to 4096, K = 24 to 6100, 0.4
// to 40 % dense, N = 16 to 33000; uniform, lognormal, banded and block-structured rows, ragged N,
// convolutions): 12 % rms error (18 % with the longest program in place of the chain).  The pick's
// time is within 1-2 % of the fastest candidate's on average (22 % at worst, of banded rows), the
// noise of the single timings included.  Programs of 32 rows, streamed, only from 8 chunks of
// K up: below, their bursts of stores are what is waited for (1500 x 100 at 90 %, N = 16384: 34.8
// against 30.8 us with 16-row ones).
// All of it but staging and stores is the packing's, computed with the plan (quad_item_times): per
// call the 48 candidates take a division each.
QuadCfg choose_quads(const sdnn_plan_s* p, int N, QuadStage stage, bool cached, double* us) {
  const int64_t tiles = (N + kQuadTileCols - 1) / kQuadTileCols;
  const uint32_t cus = p->num_cus > 0 ? p->num_cus : 256;
  const int chunks = (p->K + kQuadChunk - 1) / kQuadChunk;
  const float t_stage = stage == kQuadVec ? 0.13f : stage == kQuadDword ? 0.29f : 0.20f;
  QuadCfg best{0, 1};
  float best_t = -1.0f;
  for (int i = 0; i < p->nquads; ++i) {
    const DevQuads& d = p->quads[i];
    if (d.cap == 8 && chunks < 8 && !cached) continue;
    const float store = (d.cap == 8 ? 0.0054f : 0.0071f) * (cached ? 1.33f : 1.0f) * 4.0f * d.cap;
    for (int w = 1; w <= std::min(kMaxQuadWaves, d.nprogs); ++w) {
      const int64_t items = tiles * d.n_rb[w];
      // (32-bit divisions where they do)
      const int64_t rounds = items < (int64_t)1 << 31 ? ((uint32_t)items + cus - 1) / cus : (items + cus - 1) / cus;
      const int staged = rounds > 1 ? (chunks + 3) / 4 * 4 : chunks;
      const float t = rounds * (d.item_us[w] + t_stage * staged + store * w);
      if (best_t < 0.0f || t < best_t) {
        best_t = t;
        best = QuadCfg{i, w};
      }
    }
  }
  *us = best_t + 3.5;
  return best;
}

}  // namespace

void quad_item_times(DevQuads* d, int32_t K) {
  const int chunks = (K + kQuadChunk - 1) / kQuadChunk;
  const bool wide = d->cap <= 2;
  const double lat = wide ? 0.080 : 0.112, thr = (wide ? 0.039 : 0.016) * (double)d->blocks / std::max(1, d->nprogs);
  const double fixed = (wide ? 0.082 : 0.074) * chunks + (wide ? 0.21 : d->cap == 4 ? 0.17 : 0.58);
  for (int w = 1; w <= kMaxQuadWaves; ++w) {
    d->n_rb[w] = (d->nprogs + w - 1) / w;
    d->item_us[w] = (float)(lat * d->chain[w] + thr * std::max(0.25 * w, 1.0) + fixed);
  }
}

bool test_overrides() {
  for (char** e = environ; e && *e; ++e)
    if (strncmp(*e, "SDNN_", 5) == 0) return true;
  return false;
}

// Calls under the panel kernel's test overrides run on it.
bool quads_serve(const sdnn_plan_s* p, int32_t N, bool overrides) {
  if (overrides && (getenv("SDNN_FORCE_WAVES") || getenv("SDNN_FORCE_WG_PER_TILE") ||
                    getenv("SDNN_FORCE_TILE_MAJOR_WGS")))
    return false;
  return p->nquads > 0 && p->K > 0 && (uint64_t)N * 4u * 16 < ((uint64_t)1 << 31);
}

static QuadStage quad_stage(const float* B, const float* C, int32_t N) {
  return N % 4 == 0 && (((uintptr_t)B | (uintptr_t)C) & 15) == 0 ? kQuadVec : kQuadDword;
}

int quad_access(const sdnn_plan_s* p, const float* B, const float* C, int32_t N) {
  return 2 * (int)quad_stage(B, C, N) + (cached_stores(p, C, N) ? 1 : 0);
}

QuadCfg quad_shape(const sdnn_plan_s* p, const float* B, const float* C, int32_t N, bool conv, bool overrides,
                   double* us) {
  QuadCfg c = choose_quads(p, N, conv ? kQuadConv : quad_stage(B, C, N), cached_stores(p, C, N), us);
  if (!overrides) return c;
  const int cap = env_or("SDNN_FORCE_QUAD_CAP", 0), waves = env_or("SDNN_FORCE_QUAD_WAVES", 0);  // tests
  for (int i = 0; i < p->nquads; ++i)
    if (p->quads[i].cap == cap) c.pack = i;
  if (waves > 0) c.waves = waves;
  if (cap > 0 || waves > 0) *us = 0.0;
  return c;
}

int quad_waves(const sdnn_plan_s* p, const QuadCfg& cfg) {
  return std::max(1, std::min({cfg.waves, kMaxQuadWaves, p->quads[cfg.pack].nprogs}));
}

hipError_t launch_quads(const sdnn_plan_s* p, const float* B, float* C, int32_t N,
                        const float* bias, int epi, const int32_t* conv_hwn, const QuadCfg& cfg,
                        hipStream_t stream) {
  const DevQuads& d = p->quads[cfg.pack];
  const int64_t cus = p->num_cus > 0 ? p->num_cus : 256;
  const int waves = quad_waves(p, cfg);
  QuadArgs args;
  args.K = p->K;
  args.N = N;
  args.nchunks = (p->K + kQuadChunk - 1) / kQuadChunk;
  args.ring_chunks = (args.nchunks + 3) / 4 * 4;
  args.nprogs = d.nprogs;
  args.n_rb = (d.nprogs + waves - 1) / waves;
  args.n_tiles = (N + kQuadTileCols - 1) / kQuadTileCols;
  args.epi = epi;
  args.cached = cached_stores(p, C, N);
  const int64_t items = (int64_t)args.n_rb * args.n_tiles;
  if (items > (int64_t)1 << 30) return hipErrorInvalidValue;
  args.total_wg = (int32_t)std::min(items, cus);
  args.per_xcd = (args.total_wg + 7) / 8;
  const int budget = env_or("SDNN_POLL_BUDGET", kPollBudgetQuad);
  args.poll_budget = budget > 0 ? (uint32_t)budget : 0u;
  args.H = conv_hwn ? conv_hwn[0] : 0;
  args.W = conv_hwn ? conv_hwn[1] : 0;
  args.NB = conv_hwn ? conv_hwn[2] : 0;
  const int grid = args.per_xcd * 8;
  if (conv_hwn) return launch_stage<kQuadConv>(d, B, C, bias, args, waves, grid, stream);
  return quad_stage(B, C, N) == kQuadVec
             ? launch_stage<kQuadVec>(d, B, C, bias, args, waves, grid, stream)
             : launch_stage<kQuadDword>(d, B, C, bias, args, waves, grid, stream);
}

}  // namespace sdnn
