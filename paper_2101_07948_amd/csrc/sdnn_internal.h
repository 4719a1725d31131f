// Internal declarations shared by the host-side plan code and the HIP kernels.
// Not part of the public ABI (see include/sdnn.h).
#ifndef SDNN_INTERNAL_H_
#define SDNN_INTERNAL_H_

#include <hip/hip_runtime.h>
#include <stdint.h>

#include <vector>

#include "../../include/sdnn.h"

namespace sdnn {

// Rows of B per LDS staging slot (the paper's split-K tiling of the dense operand,
// Sec. 3.2.2) and slots in the workgroup's LDS ring.  Chunk c of B (rows
// [c*kChunk, (c+1)*kChunk)) lives in slot c % kRing while it is in use.
constexpr int kChunk = 32;
constexpr int kRing = 4;
// Stream entries are consumed in groups of kGroup: one group is 64 bytes, one scalar
// load and one scalar-cache line.
constexpr int kGroup = 8;
// Columns of C per workgroup tile: 64 lanes x 4 consecutive columns; or, for the
// 128-column tiles, 64 lanes x 2 (the narrow layout, two workgroups per CU).
constexpr int kTileCols = 256;
constexpr int kNarrowTileCols = 128;
// Zero groups appended after the last panel: the kernel's stream prefetch may read
// this many groups past the end of a panel's stream.
constexpr int kTailGroups = 16;
// Fields of a group's address words a_0..a_7 (see Packed); L = kGroup - 1.
constexpr int kRowBits = 8;         // a_j & 0xff: row inside the panel
constexpr int kEndBit = 9;          // a_L: last group of the panel
constexpr int kRingRowShift = 10;   // (a_j >> 10) & 0x7f: row of the LDS ring
constexpr int kSyncBit = 17;        // a_L: publish progress / check readiness first
constexpr int kLoShift = 17;        // a_{L-1} >> 17: lowest chunk the group reads
constexpr int kHiShift = 18;        // a_L >> 18: highest chunk the group reads
constexpr int kLoWord = kGroup - 2, kHiWord = kGroup - 1;
constexpr int kMaxChunks = 1 << 14; // chunk numbers must fit a3's high bits
// The stream of the 128-column tiles carries the same groups with 512-byte ring rows:
// the ring-row field one bit lower and the end flag at bit 8 (narrow_stream).
constexpr int kRingRowShiftNarrow = 9;  // (a_j >> 9) & 0x7f
constexpr int kEndBitNarrow = 8;
// A row of B or C must stay below 2^31 bytes (N < 2^29): the staging and the stores
// address within a row with 32-bit byte offsets.
constexpr int64_t kMaxRowBytes = (int64_t)1 << 31;
static_assert(kRing * kChunk <= 128, "ring rows must fit 7 bits");

// Host-side packed form of W in the kernel's traversal order (Sec. 3.2.2: each
// matrix stored in its own format, read sequentially).
//
//   Panels of RW consecutive rows of the permuted matrix.  A panel's entries are
//   ordered by K-chunk, then by row inside the panel, then by column, and cut into
//   groups of kGroup.  A group never spans more than kRing chunks: the entry that
//   would make it do so starts a new group, and a group cut short this way or by the
//   end of the panel is filled with zero-weight copies of its first entry.  A group
//   is 2*kGroup dwords: the kGroup fp32 weight bits, then kGroup words
//       a_j = ((c_j % kRing) * kChunk + col_j - c_j * kChunk) << 10 | row_j
//   (c_j = chunk of the entry; the shifted part is the entry's B row in the LDS
//   ring) with extra fields in the last two words
//       a6 |= c_lo << 17, a7 |= c_hi << 18 | sync << 17 | end << 9
//   where c_lo / c_hi are the lowest / highest chunk the group reads, end marks the
//   panel's last group and sync is set on a panel's first and last groups and
//   whenever c_lo or c_hi differs from the previous group's.  Panels are stored back
//   to back; panel_start holds each panel's first group (-1: the panel has no
//   entries).  The stream ends with kTailGroups zero groups.
//
//   K-segments (split_chunks = S > 0): chunks [s*S, (s+1)*S) form segment s, no group
//   holds entries of two segments (an entry of the next segment starts a new group,
//   like one too far ahead), so each segment's first group carries the sync bit (its
//   c_lo differs from the previous group's), and seg_start[p][s] is the panel's first
//   group in segment s (-1: none).  A launch may then give each run of consecutive
//   segments to its own workgroup, which starts at the run's first group and stops at
//   the first sync group whose c_lo lies past the run.
struct Packed {
  int32_t M = 0, K = 0, RW = 0, nchunks = 0, npanels = 0;
  int64_t nnz = 0, stored = 0;     // structural entries, stored entries (with padding)
  std::vector<int32_t> perm;        // [M]   original row at permuted position (reported order)
  std::vector<int32_t> panel_rows;  // [npanels*RW] original row or -1 (padding), in the
                                    // grouping order (the row order, or balanced panels)
  std::vector<int32_t> panel_out;   // [npanels*RW] row of C each panel row is stored to
                                    // (its original row, or its position in perm for
                                    // out_permuted plans), -1 for padding
  int32_t grouping = 1;             // 1: panels are consecutive rows of perm; 2: balanced
  int32_t out_permuted = 0;         // panel_out holds positions in perm
  std::vector<int32_t> panel_start; // [npanels] first group of the panel, or -1
  std::vector<int32_t> panel_order; // [npanels] panels by stored groups, heaviest first
  std::vector<uint32_t> entries;    // [2*(stored + kTailGroups*kGroup)] dwords
  double rho = 1.0;                 // nnz / sum_p |union of the panel's column sets|
  int32_t split_chunks = 0;         // chunks per K-segment (0: one segment, no table)
  int32_t nseg = 1;                 // K-segments
  std::vector<int32_t> seg_start;   // [npanels*nseg] (split_chunks > 0 only)
};

// Panel heights of the packings a default plan holds (in this order): short panels keep
// enough waves busy when a tile has few rows per CU; taller ones carry more entries per
// K-chunk (so a group spans fewer chunks of the ring) and stage each B tile for more rows.
// The fifth, 32-row panels, serves 128-column tiles only (a plan holds it when it holds
// their stream): 14 such panels share each staged B row.  The launch picks one per call
// (choose_packing).
constexpr int kShortPanel = 4, kTallPanel = 12, kMidPanel = 8, kTallestPanel = 16;
constexpr int kDeepPanel = 32;
constexpr int kMaxPackings = 5;

// ---- row quads (spmm_quad_kernel) --------------------------------------------------------
// Tile width, rows of B per chunk, chunks in the LDS ring, bytes of a staged B row (one tile
// wide), and producer waves.
constexpr int kQuadTileCols = 64;
constexpr int kQuadChunk = 64, kQuadRing = 8;
constexpr int kQuadRowBytes = 4 * kQuadTileCols;
constexpr int kQuadProducers = 4, kMaxQuadWaves = 16 - kQuadProducers;  // consumer waves
// Ring slot s at LDS address quad_slot(s): slots s and s + 4 differ in one address bit, so an
// item whose first chunk falls on slot 4 reads the stream's addresses with that bit flipped, and
// an item's chunks need only be rounded up to half the ring (rounded up to the ring, the 12
// chunks of K = 768 took 16 chunk numbers, a third of the lookahead from one item into the
// next: 3072 x 768 at 97 %, N = 16384, no activation 91.5 -> 86.9 us).
constexpr uint32_t kQuadFlip = kQuadChunk * kQuadRowBytes;
constexpr uint32_t quad_slot(uint32_t s) { return s % 4 * (2 * kQuadFlip) + s / 4 % 2 * kQuadFlip; }
// LDS address of the row of zeros that filler entries read; a second one at kQuadZeroRow ^
// kQuadFlip
constexpr int kQuadZeroRow = kQuadRing * kQuadChunk * kQuadRowBytes;
static_assert(kQuadRing == 8 && (kQuadZeroRow & kQuadFlip) == 0, "flip layout");
inline uint32_t quad_address(int32_t k) {  // of row k of B in the stream
  return quad_slot((uint32_t)k / kQuadChunk % kQuadRing) + (uint32_t)k % kQuadChunk * kQuadRowBytes;
}
// Chunks a block may span at most (quad_window picks by density): a wider window costs less
// filler but leaves fewer chunks of the ring free for DMAs in flight.
constexpr int kQuadMaxWindow = kQuadRing - 2;
constexpr int kQuadUnits = 8;           // quad-steps of a block
constexpr int kQuadTailBlocks = 8;      // zero blocks after the last program
constexpr int kQuadLoShift = 6, kQuadHiShift = 19;      // descriptor fields
constexpr uint32_t kQuadMaxBlocks = 0x3f, kQuadLoMask = 0x1fff;
constexpr uint32_t kQuadMoreDescs = 1u << kQuadLoShift;  // 64th descriptor: load the next 64
constexpr int kQuadCaps[] = {1, 2, 4, 8};  // the packings' largest programs, in quads
constexpr int kQuadPackings = 4, kQuadMaxCap = 8;
static_assert(kQuadMaxWindow <= kQuadRing, "ring too short");

// Host-side form of W for the row-quad kernel.  Rows, sorted by nonzeros (descending), form
// programs of NS quads of four rows: the most quads of 1, 2, 4, 8 up to the packing's cap for
// which the program is no longer than kQuadSlack times cap quads of average rows, so that the
// programs carry about equal work whatever the rows' lengths (a program is as long as NS times
// its longest row).  A program's entries are cut into blocks of 8 / NS steps; a step holds
// one entry of each row, or a filler (weight 0, the row of zeros), each row's entries in
// ascending column order.  While the program's lowest unread chunk is c, a block takes no
// entry from chunk c + window or above (a row that far ahead of the program's slowest one gets
// fillers).  Descriptors (one dword, see kQuadLoShift; a zero dword ends a program, every 64th
// is kQuadMoreDescs) cover runs of blocks of one lowest chunk that span at most one chunk
// more than the first of them.  A block is 64 dwords: with NS <= 2, dword 16 r + u is the
// weight of row r of set u % NS (of four rows) in step u / NS, u < 8, and dword 16 r + 8 + u its
// LDS address quad_address(k); with NS >= 4, dword 4 r + 2 u is
// the weight of row r of set u % (NS / 4) (of 16 rows) in step u / (NS / 4), u < 2, and dword
// 4 r + 2 u + 1 its LDS address.
inline int quad_dword(int NS, int j, int s) {  // of row j's weight in step s; see above
  if (NS <= 2) return 16 * (j % 4) + s * NS + j / 4;
  return 4 * (j % 16) + 2 * (s * (NS / 4) + j / 16);
}
inline int quad_addr_at(int NS) { return NS <= 2 ? 8 : 1; }  // the address's dword past it
struct QuadProgram {
  int32_t start;  // first block, or -1 (no entries)
  int32_t desc;   // first descriptor
  int32_t NS;     // quads
  int32_t blocks;
};
struct QuadPacked {
  int32_t cap = 0, nprogs = 0;
  std::vector<QuadProgram> progs;    // [nprogs], longest first
  std::vector<int32_t> rows;         // [nprogs*cap*4] original row, or -1
  std::vector<int32_t> outs;         // [nprogs*cap*4] row of C, or -1
  std::vector<uint32_t> stream;      // [64 * (blocks + kQuadTailBlocks)]
  std::vector<uint32_t> descs;       // padded with 64 zeros (the wave loads 64 at a time)
};
// Without slack the rows a little above the average halve their program, and with too much the longest
// rows set the pace of a launch.  At 1.0, 1.2, 1.4, 2 and 4: 768 x 3072 at 90 %, N = 4096: 57.3, 46.8,
// 46.8, 46.7, 46.7 us; 3072 x 768 of lognormal rows at 94 %: 46.4, 41.5, 44.1, 52.0, 64.5.
constexpr double kQuadSlack = 1.4;

// Packs W (validated CSR); out_row[i] is the row of C that row i is stored to.  False, with *out
// left empty, once the stream takes more than max_bytes.
bool pack_quads(const int32_t* row_ptr, const int32_t* col_idx, const float* values, int32_t M,
                int32_t K, int32_t cap, const int32_t* out_row, int64_t max_bytes, QuadPacked* out);
// The bytes a packing may take in a plan whose panel packings take panel_bytes; one that needs
// more is left out of the plan.  A block is 256 bytes however few entries it holds, so rows whose
// entries lie far apart in K, from one another or from the other rows', fill the stream with
// filler: 4096 rows of 16 neighbouring entries each, scattered over K = 8000, take 28, 49, 77 and
// 108 bytes an entry in the four packings (768 x 3072 at 90 %: 8.5) against 83 of the panel
// packings, and the last three are left out.
// Uniform rows of few entries keep all (4096 x 524288 at 99.99 %: 125 to 225 bytes an entry
// against 556 of the panel packings; N = 64: 1.44 ms, on the panel kernel 3.43).
inline int64_t quad_max_bytes(int64_t panel_bytes) {
  return panel_bytes / 2 > (1 << 20) ? panel_bytes / 2 : 1 << 20;
}
// Walks the packed form and checks that every entry appears once, in its row, in ascending
// column order, with unchanged bits, within the window its descriptor states.
bool check_quads(const int32_t* row_ptr, const int32_t* col_idx, const float* values, int32_t M,
                 int32_t K, const int32_t* out_row, const QuadPacked& Q);

// The program that consumer wave `stratum` of row-block rb runs (n_rb row-blocks): the strata of
// the list sorted by length in snake order over the row-blocks.
inline int quad_program(int stratum, int rb, int n_rb) {
  return stratum * n_rb + ((stratum & 1) ? n_rb - 1 - rb : rb);
}
// chain[w], w = 1 to kMaxQuadWaves: the blocks a workgroup of w consumer waves goes through one
// after another (mean over a few row-blocks).  The ring couples the waves: over a span of
// kQuadRing chunks they take as long as the slowest of them has to do there, so it is the sum over
// the spans of the most blocks any of the waves has in it.  Uniform rows make it 1.0-1.2 times the
// longest program; where the waves' rows have their entries in different parts of K, up to w times.
void quad_chains(const QuadPacked& Q, int32_t K, float* chain);

// One quad packing in device memory.
struct DevQuads {
  int32_t cap = 0, nprogs = 0;
  int64_t blocks = 0;   // of all programs
  float chain[kMaxQuadWaves + 1] = {};  // quad_chains
  // by waves: row-blocks, and what the launch model charges an item whatever the call (see
  // choose_quads): microseconds but for staging and stores
  int32_t n_rb[kMaxQuadWaves + 1] = {};
  float item_us[kMaxQuadWaves + 1] = {};
  const uint32_t* stream = nullptr;
  const uint32_t* descs = nullptr;
  const QuadProgram* progs = nullptr;
  const int32_t* rows = nullptr;
  const int32_t* outs = nullptr;
};

// The same of a panel packing: chain[w], w = 1 to kMaxPanelWaves, in groups, over spans of kRing
// chunks, for workgroups of w panels in workgroup order.
constexpr int kMaxPanelWaves = 14;
void panel_chains(const Packed& P, float* chain);

// CSR validation; returns SDNN_OK or SDNN_ERR_*.
sdnn_status validate_csr(const int32_t* row_ptr, const int32_t* col_idx, int32_t M, int32_t K);
// Algorithm 1 on 64-bit column bitsets (inputs already validated).
sdnn_status reorder_bitset(const int32_t* row_ptr, const int32_t* col_idx, int32_t M, int32_t K,
                           int32_t* perm_out);
// Builds the packed stream (inputs already validated): panel p holds rows
// group[p*RW .. p*RW+RW-1] (group is a permutation of 0..M-1; out->perm is left to the
// caller).
sdnn_status pack(const int32_t* row_ptr, const int32_t* col_idx, const float* values, int32_t M,
                 int32_t K, int32_t RW, const int32_t* group, int32_t split_chunks, Packed* out);

// The stream of the 128-column tiles: each address word a_j of P.entries re-encoded with
// the ring row at bit kRingRowShiftNarrow and the end flag at kEndBitNarrow (weights,
// row, chunk and sync fields unchanged).
std::vector<uint32_t> narrow_stream(const std::vector<uint32_t>& entries);
// True if `narrow` is narrow_stream(entries) field by field (decoded independently).
bool check_narrow_stream(const std::vector<uint32_t>& entries, const std::vector<uint32_t>& narrow);

// Staging kinds of the row-quad kernel: 16-byte pieces and stores (N % 4 == 0, B and C 16-byte
// aligned), 4-byte ones (any N), and the virtual B of a 3x3 convolution (16-byte pieces of an
// IC x H x W x NB input).
enum QuadStage { kQuadVec = 0, kQuadDword = 1, kQuadConv = 2 };
// Launch of the row-quad kernel: packing (index into sdnn_plan_s::quads), consumer waves.
struct QuadCfg {
  int32_t pack = 0, waves = 0;
};

// A launch shape sdnn_plan_tune measured fastest for one N: which packing, how many
// consumer waves per workgroup and which tile width; and, for plans with K-segments, the
// workgroups along K and the tile width of the fastest K-split call (0: not measured).  The
// panel shape is recorded also where the row-quad kernel was faster.  Which kernel was, and its
// launch, hold for calls that stage B and store C as the timed ones did (quad_access).
struct TunedShape {
  int32_t N = 0, pack = 0, waves = 0, tile = 256, splits = 0, split_tile = 0;
  int32_t quads = 0;  // the row-quad launch `quad` was faster than the panel shape
  int32_t access = 0;  // quad_access of the timed B and C
  QuadCfg quad;
};
constexpr int kTunedSlots = 8;

// One packing of the plan in device memory.
struct DevPacking {
  int32_t RW = 0, npanels = 0;
  double rho = 1.0, fill = 1.0;
  int64_t groups = 0;                     // stored groups of all panels
  float chain[kMaxPanelWaves + 1] = {};   // panel_chains (plans with uneven_chains)
  const uint32_t* entries = nullptr;      // [2*(stored + kTailGroups*kGroup)] dwords
  const uint32_t* entries_n = nullptr;    // the same groups for 128-column tiles (or null)
  const int32_t* panel_start = nullptr;   // [npanels] (in groups, -1: empty panel)
  const int32_t* panel_rows = nullptr;    // [npanels*RW] original rows (bias)
  const int32_t* panel_out = nullptr;     // [npanels*RW] rows of C the panel rows go to
  const int32_t* seg_start = nullptr;     // [npanels*nseg] in slot order (split plans)
  int32_t nseg = 1;                       // K-segments
  // (panel_start, panel_rows and panel_out are uploaded in slot order: slot j holds the
  // j-th heaviest panel; workgroups take consecutive slots)
};

}  // namespace sdnn

// The plan handle.
struct sdnn_plan_s {
  int device = -1;
  int num_cus = 0;
  int32_t M = 0, K = 0, nchunks = 0;
  int64_t nnz = 0, packed_bytes = 0;
  std::vector<int32_t> perm;
  void* d_mem = nullptr;       // one device allocation holding every packing's arrays
  int npack = 0;               // 1 (explicit panel height), 4 (short, tall, mid, tallest) or
                               // 5 (and deep, with the 128-column stream)
  int32_t out_permuted = 0;    // C rows stored in the permuted order
  int32_t in_permuted = 0;     // W's columns renamed to a caller-given order of B's rows
  int32_t split_chunks = 0;    // chunks per K-segment (0: the packings have one segment)
  int32_t grouping = 1;        // panel grouping the packings use (1: perm order, 2: balanced)
  int32_t tile_cols = 0;       // 0: the launch picks 256 or 128 columns per tile; else fixed
  const int32_t* d_perm = nullptr;  // [M] perm on the device (K-segmented plans only)
  sdnn::DevPacking pk[sdnn::kMaxPackings];
  int nquads = 0;              // quad packings (default plans: panel_rows = 0, tile_cols = 0)
  sdnn::DevQuads quads[sdnn::kQuadPackings];
  int64_t quad_bytes = 0;      // of their device memory
  bool uneven_chains = false;  // a launch of the row-quad kernel may be uneven (quads_uneven)
  sdnn::TunedShape tuned[sdnn::kTunedSlots];  // filled by sdnn_plan_tune
  int32_t ntuned = 0;
};

namespace sdnn {
// Kernel launchers (sdnn_kernels.hip).  Arguments are already checked.
hipError_t launch_spmm(const sdnn_plan_s* p, const float* B, float* C, int32_t N,
                       const float* bias, int epi, hipStream_t stream);
hipError_t launch_conv3x3(const sdnn_plan_s* p, const float* X, float* C, int32_t H, int32_t W,
                          int32_t NB, const float* bias, int epi, hipStream_t stream);
// K-split variants: `splits` workgroups along K (0: the library's choice; clamped to
// 1..nseg, nseg = p->pk[0].nseg), ws holds at least nseg * M * N floats; with one
// workgroup along K they are the plain launches and ws is not touched.
hipError_t launch_spmm_split(const sdnn_plan_s* p, const float* B, float* C, int32_t N,
                             const float* bias, int epi, int splits, float* ws,
                             hipStream_t stream);
hipError_t launch_conv3x3_split(const sdnn_plan_s* p, const float* X, float* C, int32_t H,
                                int32_t W, int32_t NB, const float* bias, int epi, int splits,
                                float* ws, hipStream_t stream);
// Workgroups along K that launch_spmm_split runs for `splits` (0: the library's
// choice) at N; 1 for a plan without K-segments (host only).
int split_runs(const sdnn_plan_s* p, int32_t N, int32_t splits);
// The non-allocating K-split call keeps its partial products in a fixed device array of
// kScratchFloats floats per device; scratch_address gives its address on `device`,
// which must be the current device (looked up once per device, then cached).
constexpr int64_t kScratchFloats = (int64_t)16 << 20;  // 64 MiB
constexpr int kMaxScratchDevices = 64;
hipError_t scratch_address(int device, float** out);
// The packing height, consumer waves and tile width launch_spmm uses at N for B and C
// that allow 16-byte staging (host only).
void launch_shape(const sdnn_plan_s* p, int32_t N, int32_t* panel_rows, int32_t* waves,
                  int32_t* tile_cols);
// Times every candidate launch shape of the plan at N on the given buffers (blocking)
// and records the fastest in p->tuned.
hipError_t tune_spmm(sdnn_plan_s* p, const float* B, float* C, int32_t N, hipStream_t stream,
                     TunedShape* chosen);
// The row-quad launch of a product at N columns (rows of the packing's largest programs and
// consumer waves; 0 and 0 where the product runs on the panel kernel).
void launch_quad_shape(const sdnn_plan_s* p, int32_t N, int32_t* program_rows, int32_t* waves);
// The row-quad kernel (sdnn_quad.hip): whether it can serve the plan's calls at N columns, the
// launch it picks at N with the microseconds its model gives that (0 for a forced one), the
// consumer waves a launch has, and its launch (conv_hwn: H, W and the images of a 3x3 convolution
// whose input is B, or null).
int quad_waves(const sdnn_plan_s* p, const QuadCfg& cfg);
// How the kernel reads B and writes C (16- or 4-byte pieces, streamed or through the caches),
// which their alignment decides.
int quad_access(const sdnn_plan_s* p, const float* B, const float* C, int32_t N);
// (overrides: any environment variable of the tests is set, so that calls without one look for
// them once)
bool test_overrides();
bool quads_serve(const sdnn_plan_s* p, int32_t N, bool overrides);
QuadCfg quad_shape(const sdnn_plan_s* p, const float* B, const float* C, int32_t N, bool conv, bool overrides,
                   double* us);
void quad_item_times(DevQuads* d, int32_t K);  // fills n_rb and item_us
// Whether a workgroup's chain of blocks is far longer than a wave's share of W (32 entries a
// block): filler, and waves that wait for one another.  Below 1.9 times the panel kernel was never
// the faster one by more than 5 % in the measurements below on_quads; uniform rows of 2 % and more
// have 1.0-1.6.
inline bool quads_uneven(const DevQuads& d, int waves, int64_t nnz) {
  return d.chain[waves] * 32.0 * d.nprogs > 1.9 * (double)nnz;
}
hipError_t launch_quads(const sdnn_plan_s* p, const float* B, float* C, int32_t N,
                        const float* bias, int epi, const int32_t* conv_hwn, const QuadCfg& cfg,
                        hipStream_t stream);
hipError_t launch_dense(const float* W, const float* B, float* C, int32_t M, int32_t K, int32_t N,
                        const float* bias, int epi, hipStream_t stream);
}  // namespace sdnn

#endif  // SDNN_INTERNAL_H_
