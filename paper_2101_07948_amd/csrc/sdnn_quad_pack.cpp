// Preparation for the row-quad kernel (SparseDNN, arXiv 2101.07948, Sec. 3.2.2: each
// matrix repacked in its kernel's traversal order): programs of row quads, their blocks and
// their descriptors (see QuadPacked).
#include <string.h>

#include <algorithm>

#include "sdnn_internal.h"

namespace sdnn {

// Chunks a block may span: enough that rows of one length seldom wait for one another.  The
// columns of a row's n-th entries scatter by about sqrt(n (1 - d)) / d across the rows, so the
// window follows the density d; past the width that keeps filler under a few per cent, a
// narrower one leaves more of the ring to the DMAs in flight.  Microseconds at windows of 2 to 6
// chunks: 3072 x 768 at 3 % (N = 16384) 114, 105, 101, 98, 96; at 6 %, lognormal 50.5, 46.2, 44.2,
// 43.8, 44.1; 768 x 3072 at 10 % (N = 4096) 51.3, 48.3, 46.8, 46.4, 46.7; 997 x 1531 at 15 % in
// 4-byte pieces 18.7, 18.9, 19.6, 20.1, 20.9; 2048 x 2048 at 30 % 36.4, 35.5, 35.3, 35.3, 35.4.
static int quad_window(const int32_t* row_ptr, int32_t M, int32_t K) {
  const double d = (double)row_ptr[M] / ((double)std::max(M, 1) * std::max(K, 1));
  return d >= 0.2 ? kQuadMaxWindow - 3 : d >= 0.08 ? kQuadMaxWindow - 2 : kQuadMaxWindow;
}

bool pack_quads(const int32_t* row_ptr, const int32_t* col_idx, const float* values, int32_t M,
                int32_t K, int32_t cap, const int32_t* out_row, int64_t max_bytes, QuadPacked* out) {
  QuadPacked& Q = *out;
  Q = QuadPacked();
  Q.cap = cap;
  // rows by nonzeros, descending, ties by index (counting sort)
  std::vector<int32_t> first((size_t)K + 2, 0), order((size_t)M);
  for (int32_t i = 0; i < M; ++i) ++first[(size_t)(K - (row_ptr[i + 1] - row_ptr[i])) + 1];
  for (size_t k = 1; k < first.size(); ++k) first[k] += first[k - 1];
  for (int32_t i = 0; i < M; ++i) order[first[(size_t)(K - (row_ptr[i + 1] - row_ptr[i]))]++] = i;

  const int window = quad_window(row_ptr, M, K);
  const double longest = kQuadSlack * cap * (double)row_ptr[M] / (double)std::max(M, 1);
  std::vector<QuadProgram> progs;
  std::vector<int32_t> prog_row;  // first row (position in order) of each program
  Q.stream.reserve((size_t)(row_ptr[M] / 4 + (int64_t)M) * 10);
  for (int32_t i0 = 0; i0 < M;) {
    int32_t NS = cap;
    while (NS > 1 && (double)NS * (row_ptr[order[i0] + 1] - row_ptr[order[i0]]) > longest) NS /= 2;
    const int RW = 4 * NS, steps = kQuadUnits / NS, to_addr = quad_addr_at(NS);
    int dword[4 * kQuadMaxCap], next_step = NS <= 2 ? NS : NS / 2;  // row j's weight: step 0, and on
    uint32_t filler[64] = {};  // a block without entries
    for (int j = 0; j < RW; ++j) {
      dword[j] = quad_dword(NS, j, 0);
      for (int st = 0; st < steps; ++st) filler[quad_dword(NS, j, st) + to_addr] = kQuadZeroRow;
    }
    // next entry, end and column of the next entry (past all columns: none left) of each row
    int32_t at[4 * kQuadMaxCap], end[4 * kQuadMaxCap], col[4 * kQuadMaxCap];
    bool any = false;
    for (int j = 0; j < RW; ++j) {
      at[j] = end[j] = 0;
      if (i0 + j < M) {
        at[j] = row_ptr[order[i0 + j]];
        end[j] = row_ptr[order[i0 + j] + 1];
      }
      col[j] = at[j] < end[j] ? col_idx[at[j]] : INT32_MAX;
      any |= at[j] < end[j];
    }
    QuadProgram P{-1, (int32_t)Q.descs.size(), NS, 0};
    if (any) {
      P.start = (int32_t)(Q.stream.size() / 64);
      int32_t lo = -1, hi = 0, top = 0;
      uint32_t n = 0;  // the open descriptor: lowest chunk, highest allowed and seen, blocks
      auto push = [&](uint32_t d) {
        if ((Q.descs.size() - (size_t)P.desc) % 64 == 63) Q.descs.push_back(kQuadMoreDescs);
        Q.descs.push_back(d);
      };
      auto close = [&] {
        push((uint32_t)top << kQuadHiShift | (uint32_t)lo << kQuadLoShift | n);
        n = 0;
      };
      for (;;) {
        int32_t low = INT32_MAX;  // the program's lowest unread column
        for (int j = 0; j < RW; ++j) low = std::min(low, col[j]);
        if (low == INT32_MAX) break;
        const int32_t clo = low / kQuadChunk;
        const int32_t limit = (clo + window) * kQuadChunk;  // first column not taken
        int32_t high = low;
        const size_t base = Q.stream.size();
        if ((int64_t)base * 4 >= max_bytes) {
          Q = QuadPacked();
          return false;
        }
        Q.stream.insert(Q.stream.end(), filler, filler + 64);
        uint32_t* blk = Q.stream.data() + base;
        for (int j = 0; j < RW; ++j) {
          uint32_t* to = blk + dword[j];
          int32_t e = at[j], k = col[j];
          for (int st = 0; st < steps && k < limit; ++st, to += next_step) {
            memcpy(to, &values[e], 4);
            to[to_addr] = quad_address(k);
            high = std::max(high, k);
            k = ++e < end[j] ? col_idx[e] : INT32_MAX;
          }
          at[j] = e;
          col[j] = k;
        }
        const int32_t chi = high / kQuadChunk;
        if (n > 0 && (clo != lo || chi > hi || n == kQuadMaxBlocks)) close();
        if (n == 0) {
          lo = clo;
          hi = chi + 1;
          top = chi;
        }
        top = std::max(top, chi);
        ++n;
        ++P.blocks;
      }
      close();
      push(0);
    }
    progs.push_back(P);
    prog_row.push_back(i0);
    i0 += RW;
  }
  Q.stream.resize(Q.stream.size() + (size_t)kQuadTailBlocks * 64, 0u);
  Q.descs.resize(Q.descs.size() + 64, 0u);

  // the program table, longest first (ties in packing order)
  Q.nprogs = (int32_t)progs.size();
  std::vector<int32_t> by((size_t)Q.nprogs);
  for (int32_t p = 0; p < Q.nprogs; ++p) by[p] = p;
  std::stable_sort(by.begin(), by.end(),
                   [&](int32_t x, int32_t y) { return progs[x].blocks > progs[y].blocks; });
  Q.rows.assign((size_t)Q.nprogs * cap * 4, -1);
  Q.outs.assign((size_t)Q.nprogs * cap * 4, -1);
  for (int32_t p = 0; p < Q.nprogs; ++p) {
    const QuadProgram& P = progs[by[p]];
    Q.progs.push_back(P);
    for (int j = 0; j < 4 * P.NS && prog_row[by[p]] + j < M; ++j) {
      const int32_t row = order[prog_row[by[p]] + j];
      Q.rows[(size_t)p * cap * 4 + j] = row;
      Q.outs[(size_t)p * cap * 4 + j] = out_row[row];
    }
  }
  return true;
}

void quad_chains(const QuadPacked& Q, int32_t K, float* chain) {
  const int spans = std::max(0, K - 1) / (kQuadChunk * kQuadRing) + 1;
  std::vector<int32_t> most(spans), own(spans);
  for (int w = 1; w <= kMaxQuadWaves; ++w) {
    const int n_rb = (Q.nprogs + w - 1) / w, step = std::max(1, n_rb / 4);
    double sum = 0.0;
    int looked_at = 0;
    for (int rb = 0; rb < n_rb; rb += step, ++looked_at) {
      std::fill(most.begin(), most.end(), 0);
      for (int s = 0; s < w; ++s) {
        const int p = quad_program(s, rb, n_rb);
        if (p >= Q.nprogs || Q.progs[p].start < 0) continue;
        std::fill(own.begin(), own.end(), 0);
        for (size_t d = (size_t)Q.progs[p].desc; Q.descs[d] != 0; ++d)
          if (Q.descs[d] != kQuadMoreDescs)
            own[(Q.descs[d] >> kQuadLoShift & kQuadLoMask) / kQuadRing] += (int32_t)(Q.descs[d] & kQuadMaxBlocks);
        for (int b = 0; b < spans; ++b) most[b] = std::max(most[b], own[b]);
      }
      for (int b = 0; b < spans; ++b) sum += most[b];
    }
    chain[w] = looked_at ? (float)(sum / looked_at) : 0.0f;
  }
}

void panel_chains(const Packed& P, float* chain) {
  const int spans = std::max(1, (P.nchunks + kRing - 1) / kRing);
  std::vector<int32_t> most(spans), own(spans);
  for (int w = 1; w <= kMaxPanelWaves; ++w) {
    const int n_rb = (P.npanels + w - 1) / w, step = std::max(1, n_rb / 4);
    double sum = 0.0;
    int looked_at = 0;
    for (int rb = 0; rb < n_rb; rb += step, ++looked_at) {
      std::fill(most.begin(), most.end(), 0);
      for (int j = rb * w; j < std::min((rb + 1) * w, P.npanels); ++j) {
        const int32_t first = P.panel_start[P.panel_order[j]];
        if (first < 0) continue;
        std::fill(own.begin(), own.end(), 0);
        for (const uint32_t* a = &P.entries[(size_t)first * 2 * kGroup + kGroup];; a += 2 * kGroup) {
          ++own[(a[kLoWord] >> kLoShift) / kRing];
          if (a[kHiWord] >> kEndBit & 1u) break;
        }
        for (int b = 0; b < spans; ++b) most[b] = std::max(most[b], own[b]);
      }
      for (int b = 0; b < spans; ++b) sum += most[b];
    }
    chain[w] = looked_at ? (float)(sum / looked_at) : 0.0f;
  }
}

bool check_quads(const int32_t* row_ptr, const int32_t* col_idx, const float* values, int32_t M,
                 int32_t K, const int32_t* out_row, const QuadPacked& Q) {
  const uint32_t last_chunk = (uint32_t)std::max(0, (K - 1) / kQuadChunk);
  const size_t blocks = Q.stream.size() / 64, stride = (size_t)Q.cap * 4;
  if (Q.cap < 1 || Q.cap > kQuadMaxCap || Q.progs.size() != (size_t)Q.nprogs) return false;
  if (Q.rows.size() != Q.nprogs * stride || Q.outs.size() != Q.rows.size()) return false;
  if (Q.stream.size() % 64 != 0 || blocks < (size_t)kQuadTailBlocks) return false;
  std::vector<char> seen((size_t)std::max(M, 1), 0);
  size_t total_blocks = 0;
  for (int32_t p = 0; p < Q.nprogs; ++p) {
    const QuadProgram& P = Q.progs[p];
    if (P.NS < 1 || P.NS > Q.cap || kQuadUnits % P.NS != 0) return false;
    if (p > 0 && P.blocks > Q.progs[p - 1].blocks) return false;
    std::vector<int32_t> at(stride, 0), end(stride, 0);
    int64_t left = 0;
    for (size_t j = 0; j < stride; ++j) {
      const int32_t row = Q.rows[p * stride + j];
      if (row < 0) {
        if (Q.outs[p * stride + j] >= 0) return false;
        continue;
      }
      if (j >= (size_t)P.NS * 4 || row >= M || seen[row]++ || Q.outs[p * stride + j] != out_row[row])
        return false;
      at[j] = row_ptr[row];
      end[j] = row_ptr[row + 1];
      left += end[j] - at[j];
    }
    if (P.start < 0) {
      if (left != 0 || P.blocks != 0) return false;
      continue;
    }
    if (left == 0) return false;
    size_t b = (size_t)P.start;
    uint32_t prev_lo = 0;
    for (size_t d = (size_t)P.desc;; ++d) {
      if (d + 64 > Q.descs.size()) return false;  // a wave may load 64 descriptors from here
      if ((Q.descs[d] == kQuadMoreDescs) != ((d - (size_t)P.desc) % 64 == 63) && Q.descs[d] != 0)
        return false;
      if (Q.descs[d] == kQuadMoreDescs) continue;
      const uint32_t n = Q.descs[d] & kQuadMaxBlocks;
      if (n == 0) {
        if (Q.descs[d] != 0) return false;
        break;
      }
      const uint32_t lo = Q.descs[d] >> kQuadLoShift & kQuadLoMask, hi = Q.descs[d] >> kQuadHiShift;
      if (hi < lo || hi - lo >= (uint32_t)kQuadMaxWindow || hi > last_chunk || lo < prev_lo) return false;
      prev_lo = lo;
      for (uint32_t i = 0; i < n; ++i, ++b) {
        if (b + kQuadTailBlocks >= blocks) return false;
        const uint32_t* blk = Q.stream.data() + 64 * b;
        for (int st = 0; st < kQuadUnits / P.NS; ++st)
          for (int j = 0; j < 4 * P.NS; ++j) {
            const int at_w = quad_dword(P.NS, j, st);
            const uint32_t w = blk[at_w], addr = blk[at_w + quad_addr_at(P.NS)];
            if (addr == (uint32_t)kQuadZeroRow) {
              if (w != 0) return false;
              continue;
            }
            if (at[j] >= end[j]) return false;
            const int32_t k = col_idx[at[j]];
            uint32_t bits;
            memcpy(&bits, &values[at[j]], 4);
            const uint32_t c = (uint32_t)(k / kQuadChunk);
            if (bits != w || addr != quad_address(k) ||
                c < lo || c > hi)
              return false;
            ++at[j];
            --left;
          }
      }
    }
    if (left != 0 || b != (size_t)P.start + P.blocks) return false;
    total_blocks += P.blocks;
  }
  for (int32_t i = 0; i < M; ++i)
    if (!seen[i]) return false;
  return total_blocks + kQuadTailBlocks == blocks;
}

}  // namespace sdnn
