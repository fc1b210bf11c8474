// encode.hip -- gfx950 kernels and host driver for PivCo-Huffman encoding.
//
// Encoding (Sec. 4 of the paper) uses the same tree as decoding and walks it
// top-down: each internal node receives the codes of the symbols passing
// through it, emits one bit per symbol (its bitmap) and partitions the
// symbols between its children (the enc_partition primitives of Table 11).
// The driver:
//   1. k_hist        symbol histogram of every block and of every slice of it
//                    (end-to-end encode time is dominated by this
//                    count, Sec. 4); k_slice_prefix turns the slice counts
//                    into per-slice prefixes;
//   2. k_code        per block: optimal length-limited lengths (package-merge,
//                    the host's tie rules) or the supplied tree, then from the
//                    lengths and the histogram canonical codes, breadth-first
//                    node table, n_v and n_right, the rANS selection rule,
//                    body sizes and offsets, and the block header bytes;
//   3. k_scan        offsets of every block's areas (exclusive scans); a call
//                    of one block finds them in k_code;
//   4. k_split       per slice of a block: per level, every wave turns 64
//                    symbols at a time of the level's array into a 64-bit
//                    ballot of code bits (LSB first = stream order) and moves
//                    them to the children's places in LDS (stable); then the
//                    nodes' bits go out word by word.
// Without entropy-coded nodes the blocks' places in the stream are known by
// then: k_head writes the headers and k_split the bodies.  With them k_split
// fills a byte-packed raw image per block and word-aligned rANS bitmaps, and
//   5. k_rans_enc    codes the chunks (32-lane interleaved binary rANS, one wave
//                    per chunk, steps in reverse order), or k_fse_enc (byte
//                    tANS);
//   6. k_sizes       block sizes from the rANS body sizes; k_scan2 the block
//                    offsets and the stream size (and the sizes of few
//                    blocks);
//   7. k_assemble    stream header, offset tables, block headers, raw images
//                    (aligned 4-byte words) and rANS bodies.
// The stream length and the call's status go to device memory with the sizes.
// Nothing waits on the host: pivco_encode_async leaves the length and status
// in device memory; pivco_encode reads them back.
#include <hip/hip_runtime.h>

#include <algorithm>
#include <cstring>
#include <vector>

#include "pivco_int.h"

namespace pivco {

bool tree_is_complete(const uint8_t len[256], uint32_t max_len);

namespace {

constexpr int kWaveE = 64;
// Symbols of a slice (a histogram row, a split workgroup).
constexpr uint32_t kSliceSmall = 1u << 12, kSliceLarge = 1u << 13;
constexpr uint32_t kHdrStride = 1216;   // block header bytes: 12 + 128 + 32 + 4 * 255 <= this
constexpr uint32_t kAsmSeg = 2048;      // output words per assembling workgroup: 8 a thread
constexpr uint32_t kTailBlocks = 64;    // blocks whose sizes and offsets one workgroup finds
constexpr uint32_t kScanNT = 1024;
// Error word of one encode (in its status area); the first error wins.
constexpr uint32_t kErrArg = 1;          // a block's tree: PIVCO_E_ARG
constexpr uint32_t kErrUnsupported = 2;  // a tANS cursor stream past its 16-bit length: PIVCO_E_UNSUPPORTED

// Per-block description for the split kernel, written by k_code.  Leaves
// are numbered in code order (of the left-justified codes), so the symbols
// that pass a node are the leaves of one interval.
struct EncBlock {
  uint64_t in_off;        // first input symbol
  uint32_t n;             // symbols
  uint32_t I;             // internal nodes (0: constant block, nothing to split)
  uint32_t maxlen;        // node levels
  uint32_t nleaf;         // symbols with a code
  uint32_t lvl[18];       // first node id of each depth
  int32_t kbase[16];      // node at depth d with code prefix p: slot p + kbase[d] (in the
                          // split kernel's tables; a prefix without a node takes one too
                          // where a flat-subtree tree has a single leaf among the nodes)
  uint8_t nfl[16];        // flat nodes per level (the level's first nodes)
  uint32_t bit[256];      // node's first bit: in the block's raw image (raw
                          // node) or in its rANS bitmap words (rANS node)
  uint32_t kind[8];       // bit i: node i is rANS-coded
  uint16_t pay[256];      // a symbol's code, left-justified in 16 bits
  uint8_t lo[256];        // node's leaves [lo, hi), those of its right child
  uint8_t mid1[256];      // [mid, hi): mid - 1 and hi - 1
  uint8_t hi1[256];
  uint8_t child[256][2];  // internal id, or 255 for a leaf
  uint8_t slot[256];      // node's slot less its id: the single leaves before it (at most 12)
  uint8_t leaf[256];      // leaf of each symbol (255, never a leaf then, without a code)
  uint8_t depth[256];     // node's level
  uint8_t fd[256];        // flat node: its depth D (>= 2), 0 for binary nodes
};
static_assert(sizeof(EncBlock) % 16 == 0, "EncBlock areas stay 16-byte aligned");
static_assert(sizeof(EncBlock) <= 4048, "a block's share of the workspace (see ws_layout)");

// Per-block layout (k_code), offsets (k_scan) and size (without entropy-coded
// nodes k_code, else k_sizes and k_scan2).
struct BlockLay {
  uint32_t n;             // symbols
  uint32_t hlen;          // header bytes
  uint32_t raw_bytes;     // raw bodies
  uint32_t ans_words;     // words its rANS nodes decode into: sum of ceil(n_v / 32)
  uint32_t n_rnodes;      // rANS-coded nodes
  uint32_t n_chunks;      // their chunks
  uint64_t slot_bytes;    // output slot bytes of its chunks
  uint64_t img_off;       // its raw image in the image area (bytes, 16-aligned); without
                          // entropy-coded nodes in the stream itself
  uint64_t rbm_off;       // its rANS bitmaps in the rANS bitmap area (words)
  uint64_t chunk0;        // its first chunk job
  uint64_t slot0;         // its first slot byte
  uint64_t ans0;          // scratch words of the blocks before it (stream table)
  uint64_t out_off;       // the block in the stream (bytes)
  uint32_t comp;          // block bytes (comp_size)
  uint32_t pad;
};

// A rANS-coded node of a block, in node order (k_code).
struct RansNode {
  uint32_t rword;         // first word of its bitmap among the block's rANS words
  uint32_t nv;            // bits
  uint32_t p1q;           // 12-bit probability of a 1 bit (ans_mode 3: the tANS marker)
  uint32_t ch0;           // its first chunk among the block's chunks
  uint64_t sl0;           // its first slot byte among the block's slots
};

struct RansJob {
  uint64_t bmp_word;      // word of the chunk's first bit in the rANS bitmap area
  uint64_t slot;          // byte offset of the chunk's output slot
  uint32_t nbits;
  uint32_t p1q;
  uint32_t block;
  uint32_t rnode;         // its node among the block's rANS nodes
  uint32_t first;         // 1: first chunk of its node
  uint32_t dst;           // byte offset of the chunk in its block (k_sizes)
};

// Batch totals (k_scan, k_scan2).
struct Totals {
  uint64_t img_bytes, rbm_words, chunks, slot_bytes, ans_words, out_bytes;
  uint64_t pad[2];
};

__device__ __forceinline__ uint32_t wave_incl_scan(uint32_t v) {
  v += static_cast<uint32_t>(__builtin_amdgcn_update_dpp(0, static_cast<int>(v), 0x111, 0xf, 0xf, false));
  v += static_cast<uint32_t>(__builtin_amdgcn_update_dpp(0, static_cast<int>(v), 0x112, 0xf, 0xf, false));
  v += static_cast<uint32_t>(__builtin_amdgcn_update_dpp(0, static_cast<int>(v), 0x114, 0xf, 0xf, false));
  v += static_cast<uint32_t>(__builtin_amdgcn_update_dpp(0, static_cast<int>(v), 0x118, 0xf, 0xf, false));
  v += static_cast<uint32_t>(__builtin_amdgcn_update_dpp(0, static_cast<int>(v), 0x142, 0xa, 0xf, false));
  v += static_cast<uint32_t>(__builtin_amdgcn_update_dpp(0, static_cast<int>(v), 0x143, 0xc, 0xf, false));
  return v;
}

__device__ __forceinline__ void wave_sync() {
  __builtin_amdgcn_fence(__ATOMIC_RELEASE, "wavefront");
  __builtin_amdgcn_wave_barrier();
  __builtin_amdgcn_fence(__ATOMIC_ACQUIRE, "wavefront");
}

// Probability of a 1 bit in 12-bit fixed point, rounded to nearest and
// clamped to [1, 4095] (the format's reading of the 12-bit binary coder).
__device__ __forceinline__ uint32_t p1q_of(uint32_t nv, uint32_t nr) {
  const uint64_t q = (static_cast<uint64_t>(nr) * 4096 + nv / 2) / nv;
  return static_cast<uint32_t>(q < 1 ? 1 : q > 4095 ? 4095 : q);
}

// The rANS selection rule: ans_mode 1 codes nodes whose one-bit fraction is
// below 0.1 or above 0.9; 2 codes every node; nodes no symbol passes never.
__device__ __forceinline__ bool select_ans(uint32_t mode, uint32_t nv, uint32_t nr) {
  if (nv == 0) return false;
  if (mode == 1) return 10ull * nr < nv || 10ull * nr > 9ull * nv;
  return mode == 2;
}

// The selection rule of the byte tANS coder (ans_mode 3, Sec. 5.2): a
// binary node of at least 256 bits whose majority bit has a fraction above
// 0.625 (8 maj > 5 n_v) takes table t = round(100 x that fraction) - 49
// (halves up, at most 50) when the table's expected bits per bitmap bit h_t
// make (depth + h_t) / (depth + 1) < 0.95; dmax[t] is the number of depths
// that pass (the test holds exactly for depth < 19 - 20 h_t).  Returns the
// marker (t, | 0x80 when 1 bits are the minority and the bitmap is coded
// complemented), or 0.
__device__ __forceinline__ uint32_t fse_marker(uint32_t nv, uint32_t nr, uint32_t depth,
                                               const uint8_t *dmax) {
  if (nv < 256 || nr > nv) return 0;
  const uint32_t zeros = nv - nr, maj = nr >= zeros ? nr : zeros;
  if (8ull * maj <= 5ull * nv) return 0;
  uint64_t pct = (200ull * maj + nv) / (2ull * nv);
  if (pct > 99) pct = 99;
  const uint32_t t = static_cast<uint32_t>(pct) - 49;
  if (depth >= dmax[t]) return 0;
  return t | (nr < zeros ? 0x80u : 0u);
}

// Output slot of a chunk of nbits bits: lane states, at most one 16-bit word
// per bit, padding.  A tANS chunk of the same bits fits too: 128 header
// bytes, per cursor at most 11 bits a byte rounded up to bytes, and padding
// come to at most 161 + 11 nbits / 64 bytes, within this size from 14 bits
// on; below that, two cursors of one step each take at most 132 bytes.
__host__ __device__ __forceinline__ uint32_t slot_size(uint32_t nbits) {
  return (kChunkHdr + 2 * nbits + 4 + 15) & ~15u;
}

// ---------------------------------------------------------------------------
// kernels
// ---------------------------------------------------------------------------
// 16 bytes at a time; n16 of them.
__device__ __forceinline__ void fill_zero16(uint4 *p, uint64_t n16, uint64_t t, uint64_t step) {
  for (uint64_t i = t; i < n16; i += step) p[i] = make_uint4(0, 0, 0, 0);
}

// Zeroes the image and rANS bitmap areas up to the sizes k_scan found (the
// split kernel ORs bits into them).  Both areas are 256-byte aligned with
// slack past their ends.
__global__ __launch_bounds__(256) void k_zero_areas(uint32_t *img, uint32_t *rbm, const Totals *tot) {
  const uint64_t t = blockIdx.x * 256ull + threadIdx.x, step = gridDim.x * 256ull;
  fill_zero16(reinterpret_cast<uint4 *>(img), (tot->img_bytes + 15) / 16, t, step);
  fill_zero16(reinterpret_cast<uint4 *>(rbm), (tot->rbm_words + 3) / 4, t, step);
}

// Histogram of every block, one workgroup per slice: the slice's counts go to
// its own row of slh (the split kernel's slices start at the same
// boundaries); a block of one slice also writes them to its row of hist
// (k_slice_prefix writes the totals of larger blocks).  Lanes of equal
// symbols count in kHistCopies places, so that a frequent symbol does not
// serialise the LDS atomics (64 MiB with one symbol at 0.9: 207 -> 31 us,
// 256 MiB Zipf 206 -> 92 us).  The call's error word and, where zero16 is
// not 0, the areas that the split kernel ORs into are cleared here too.
constexpr int kHistCopies = 16;
__global__ __launch_bounds__(256) void k_hist(const uint8_t *in, uint64_t n, uint32_t bs, uint32_t slice,
                                              uint32_t spb, uint32_t *hist, uint32_t *slh, uint32_t *err,
                                              uint4 *areas, uint64_t zero16) {
  __shared__ uint32_t h[kHistCopies][257];
  const uint32_t tid = threadIdx.x;
  if (blockIdx.x == 0 && tid == 0) *err = 0;
  fill_zero16(areas, zero16, blockIdx.x * 256ull + tid, gridDim.x * 256ull);
  for (uint32_t i = tid; i < kHistCopies * 257; i += 256) (&h[0][0])[i] = 0;
  __syncthreads();
  const uint64_t b = blockIdx.x / spb, sl = blockIdx.x % spb;
  const uint64_t bstart = b * bs;
  const uint64_t bend = bstart + bs < n ? bstart + bs : n;
  const uint64_t s0 = bstart + sl * slice;
  const uint32_t len = s0 >= bend ? 0u : bend - s0 < slice ? static_cast<uint32_t>(bend - s0) : slice;
  const uint8_t *p = in + s0;
  uint32_t *hc = h[tid % kHistCopies];
  for (uint32_t i = 16 * tid; i < len; i += 16 * 256) {
    if (i + 16 <= len) {
      uint32_t w[4];
      __builtin_memcpy(w, p + i, 16);         // no alignment
#pragma unroll
      for (int e = 0; e < 16; ++e) atomicAdd(&hc[(w[e >> 2] >> (8 * (e & 3))) & 255], 1u);
    } else {
      for (uint32_t e = i; e < len; ++e) atomicAdd(&hc[p[e]], 1u);
    }
  }
  __syncthreads();
  uint32_t v = 0;
#pragma unroll
  for (int j = 0; j < kHistCopies; ++j) v += h[j][tid];
  slh[static_cast<uint64_t>(blockIdx.x) * 256 + tid] = v;
  if (spb == 1) hist[b * 256 + tid] = v;
}

// Per block, the slice histograms become exclusive prefixes: row k holds the
// count of each symbol in the block's slices before slice k, and the block's
// row of hist the totals.  Few rows: a workgroup per block, a thread per
// symbol, 16 rows read before any is rewritten.
__global__ __launch_bounds__(256) void k_slice_prefix(uint32_t *slh, uint32_t spb, uint32_t *hist) {
  uint32_t *row = slh + static_cast<uint64_t>(blockIdx.x) * spb * 256 + threadIdx.x;
  uint32_t run = 0, k = 0;
  for (; k + 16 <= spb; k += 16) {
    uint32_t c[16];
#pragma unroll
    for (int j = 0; j < 16; ++j) c[j] = row[256ull * (k + j)];
#pragma unroll
    for (int j = 0; j < 16; ++j) {
      row[256ull * (k + j)] = run;
      run += c[j];
    }
  }
  for (; k < spb; ++k) {
    const uint32_t c = row[256ull * k];
    row[256ull * k] = run;
    run += c;
  }
  hist[static_cast<uint64_t>(blockIdx.x) * 256 + threadIdx.x] = run;
}

// Many rows (past kPrefixRows): one workgroup cannot draw a block's rows fast
// enough (1024 rows, 1 MiB: 38 us), so a block has 16 workgroups of 16
// symbols, and 64 shares of the rows in each; a share is summed, then
// rewritten from the sums of the shares before it.
constexpr uint32_t kPrefixRows = 48;
__global__ __launch_bounds__(1024) void k_slice_prefix_wide(uint32_t *slh, uint32_t spb, uint32_t *hist) {
  __shared__ uint32_t sums[64][17];
  const uint32_t b = blockIdx.x >> 4, sym = 16 * (blockIdx.x & 15) + (threadIdx.x & 15), g = threadIdx.x >> 4;
  uint32_t *row = slh + static_cast<uint64_t>(b) * spb * 256 + sym;
  const uint32_t per = (spb + 63) / 64;
  const uint32_t r0 = g * per < spb ? g * per : spb, r1 = r0 + per < spb ? r0 + per : spb;
  constexpr uint32_t kB = 16;
  uint32_t c[kB], run = 0;
  for (uint32_t r = r0; r < r1; r += kB) {
#pragma unroll
    for (uint32_t j = 0; j < kB; ++j) c[j] = r + j < r1 ? row[256ull * (r + j)] : 0u;
#pragma unroll
    for (uint32_t j = 0; j < kB; ++j) run += c[j];
  }
  sums[g][threadIdx.x & 15] = run;
  __syncthreads();
  if (threadIdx.x < 16) {
    uint32_t at = 0;
    for (uint32_t i = 0; i < 64; ++i) {
      const uint32_t v = sums[i][threadIdx.x];
      sums[i][threadIdx.x] = at;
      at += v;
    }
    hist[256ull * b + sym] = at;
  }
  __syncthreads();
  run = sums[g][threadIdx.x & 15];
  for (uint32_t r = r0; r < r1; r += kB) {
    if (per > kB) {                          // else they are still here
#pragma unroll
      for (uint32_t j = 0; j < kB; ++j) c[j] = r + j < r1 ? row[256ull * (r + j)] : 0u;
    }
#pragma unroll
    for (uint32_t j = 0; j < kB; ++j)
      if (r + j < r1) {
        row[256ull * (r + j)] = run;
        run += c[j];
      }
  }
}

// The call's result on the device: the stream length (also when it exceeds
// out_cap, in which case nothing is written) and a status.  One thread, after
// every kernel that may set the error word.
struct Result {
  uint64_t out_cap;
  uint64_t *d_len;
  int32_t *d_status;
};
__device__ void finish(uint64_t n, uint32_t *err, const Result &r) {
  const uint32_t e = atomicAdd(err, 0u);
  *r.d_len = n;
  *r.d_status = e == kErrArg ? PIVCO_E_ARG : e ? PIVCO_E_UNSUPPORTED : n > r.out_cap ? PIVCO_E_CAPACITY : PIVCO_OK;
}

// Exclusive sum over a workgroup of kScanNT threads; *all gets the sum.
__device__ __forceinline__ uint64_t block_excl_scan(uint64_t v, uint64_t *part, uint64_t *all) {
  const uint32_t wave = threadIdx.x >> 6, lane = __lane_id();
  uint64_t x = v;
#pragma unroll
  for (int o = 1; o < kWaveE; o <<= 1) {
    const uint64_t y = __shfl_up(x, o, kWaveE);
    if (lane >= static_cast<uint32_t>(o)) x += y;
  }
  if (lane == kWaveE - 1) part[wave] = x;
  __syncthreads();
  uint64_t before = 0, sum = 0;
  for (uint32_t w = 0; w < kScanNT / kWaveE; ++w) {
    const uint64_t q = part[w];
    before += w < wave ? q : 0u;
    sum += q;
  }
  *all = sum;
  __syncthreads();
  return before + x - v;
}

__host__ __device__ __forceinline__ uint64_t stream_tables(uint64_t nb) { return kHeaderBytes + 16 * (nb + 1); }

// Area of a block's raw image (16-aligned, with 16 bytes of slack) and of its
// rANS bitmap words.
__device__ __forceinline__ uint64_t img_area(const BlockLay &L) { return (static_cast<uint64_t>(L.raw_bytes) + 16 + 15) & ~15ull; }
__device__ __forceinline__ uint64_t rbm_area(const BlockLay &L) { return (static_cast<uint64_t>(L.ans_words) + 3) & ~3ull; }

// Code lengths of a block on the device (one thread per symbol), the same
// package-merge and determinism rules as the host's lengths_from_counts
// (items by weight; on equal weight a single before a package, symbols by
// id, packages in creation order; the multiset of lengths handed out again
// ascending to the symbols by (count desc, id asc)), in parallel form:
//   * the present symbols are ranked by (count, id) by counting over all 256
//     counts (broadcast LDS reads);
//   * row L holds the m singles in that order; row r - 1 merges the singles
//     with the packages (sums of consecutive pairs) of row r: single i lands
//     at i + #(packages lighter than it), package j at j + #(singles no
//     heavier), and positions past 2m - 2 are dropped.
//     Each row keeps the positions of its singles;
//   * buying the first k = 2m - 2 items of row 1 buys the singles placed
//     below k and 2 (k - singles) items of the next row, and so on; single i
//     is as deep as the rows that bought more than i singles, so the depths
//     fall with i and the symbol that is the j-th by (count desc, id asc) gets
//     the depth of single m - 1 - j.
// The rows are a chain, so their latency, not work, is the kernel's time.  A
// count over a sorted row of 256 is 16 comparisons with the last item of each
// 16 and 16 more within one: two round trips to LDS where a binary search took
// 9 (2450 -> 1270 cycles a row, the ranking 8300 -> 4500).  With few blocks a
// second half of the workgroup takes the packages and half the ranking; with
// more than two blocks a CU, work counts too and 256 threads do it all.  One
// block of 64 KiB: 17 us with the layout (24 with 256 threads and binary
// searches; one wave per block took 100 + 6); 4096 blocks 99 us with 256
// threads, 112 with 512, was 312 + 22.  W is the weights' type: a package's
// weight is at most the code length limit times the block's size, which for
// blocks below 2^24 symbols is below 2^28.
constexpr uint32_t kFewBlocks = 512;
constexpr uint32_t kTreeRows = kMaxLenGpu + 1;
struct TreeSmem {
  alignas(16) uint64_t w[256];     // counts in (count, id) order, the largest value past the last
  alignas(16) uint64_t row[2][512];   // item weights of two rows
  alignas(16) uint64_t pk[256];    // packages of the row below, the largest value past the last
  alignas(16) uint64_t wl[16], pl[16];   // the last of each 16 of w and of pk
  alignas(16) uint32_t cnt[256];   // counts by symbol
  uint16_t rank[256];              // symbols of the upper half's share ranked before this one
  alignas(16) uint16_t spos[kTreeRows][256];   // row r: position of single i (0xFFFF: not in the row)
};

// a < b as 0 or 1 for values below 2^31: the sign of the difference, as a
// comparison's mask may only be read two wait states after it is made.
template <class W>
__device__ __forceinline__ uint32_t less(W a, W b) {
  if (sizeof(W) == 4) return static_cast<uint32_t>(a - b) >> 31;
  return a < b ? 1u : 0u;
}

// The number of items of a sorted row of 256 (absent items: the largest
// value) that are less than x; pv: the last item of each run of 16.
template <class W>
__device__ __forceinline__ uint32_t row_count(const W *row, const W *pv, W x) {
  uint32_t g = 0, k = 0;
#pragma unroll
  for (uint32_t i = 0; i < 16; ++i) g += less<W>(pv[i], x);
  g = 16 * (g < 15 ? g : 15u);
#pragma unroll
  for (uint32_t i = 0; i < 16; ++i) k += less<W>(row[g + i], x);
  return g + k;
}

// A thread per symbol, single and package, or with NT = 512 two, u = thread &
// 255: the upper half takes half the ranking and the packages.  The length of
// symbol u for the threads below 256.
template <uint32_t NT, class W>
__device__ uint32_t tree_lengths(TreeSmem &sm, uint32_t m, uint32_t L, bool *bad) {
  const uint32_t u = threadIdx.x & 255, lane = __lane_id();
  const uint32_t wave = __builtin_amdgcn_readfirstlane(threadIdx.x >> 6);
  const bool upper = NT == 256 || wave >= 4, lower = NT == 256 || wave < 4;
  W *w = reinterpret_cast<W *>(sm.w), *pk = reinterpret_cast<W *>(sm.pk);
  W *wl = reinterpret_cast<W *>(sm.wl), *pl = reinterpret_cast<W *>(sm.pl);
  W *row[2] = {reinterpret_cast<W *>(sm.row[0]), reinterpret_cast<W *>(sm.row[1])};
  const W none = ~static_cast<W>(0) >> 1;
  // rank by (count, id): a smaller id goes first on the same count.  The
  // absent symbols, all lighter, are taken off again.
  const uint32_t c = sm.cnt[u];
  uint32_t rank = 0;
#pragma unroll 1
  for (uint32_t q = lower ? 0 : 2, e = upper ? 4 : 2; q < e; ++q) {
    const uint32_t *v = sm.cnt + 64 * q;
    if (q == (wave & 3)) {
#pragma unroll 16
      for (uint32_t i = 0; i < 64; ++i) rank += less<uint32_t>(v[i], c + less<uint32_t>(i, lane));
    } else {
      const uint32_t x = c + (q < (wave & 3) ? 1u : 0u);
#pragma unroll 16
      for (uint32_t i = 0; i < 64; ++i) rank += less<uint32_t>(v[i], x);
    }
  }
  if (!lower) sm.rank[u] = static_cast<uint16_t>(rank);
  __syncthreads();
  if (lower) {
    rank += (NT == 256 ? 0u : sm.rank[u]) - (256 - m);
    if (c) {
      w[rank] = c;
      row[L & 1][rank] = c;
      if ((rank & 15) == 15) wl[rank >> 4] = c;
    }
    if (u >= m) {
      w[u] = none;
      if ((u & 15) == 15) wl[u >> 4] = none;
    }
    sm.spos[L][u] = u < m ? static_cast<uint16_t>(u) : 0xFFFFu;
  }
  const uint32_t cap = 2 * m - 2;
  uint32_t rl = m, rl_l = m;               // items of row r; lane r keeps its row's
  __syncthreads();
  const W x = w[u];                        // single u
  // this symbol's run of equal counts: [lt, le)
  uint32_t lt = 0, le = 0;
#pragma unroll 1
  for (uint32_t i = 0; i < 2; ++i) {
    lt = le;
    le = row_count<W>(w, wl, c + i);
  }
  for (uint32_t r = L; r > 1; --r) {
    const W *cur = row[r & 1];
    W *nxt = row[(r - 1) & 1];
    const uint32_t np = rl / 2;
    const uint32_t total = m + np < cap ? m + np : cap;
    W y = none;
    if (upper) {
      if (u < np) y = cur[2 * u] + cur[2 * u + 1];
      pk[u] = y;
      if ((u & 15) == 15) pl[u >> 4] = y;
    }
    __syncthreads();
    if (upper) {
      const uint32_t at = u + row_count<W>(w, wl, y + 1);    // singles no heavier
      if (u < np && at < total) nxt[at] = y;
    }
    if (lower) {
      const uint32_t at = u + row_count<W>(pk, pl, x);   // packages lighter
      const bool in = u < m && at < total;
      if (in) nxt[at] = x;
      sm.spos[r - 1][u] = in ? static_cast<uint16_t>(at) : 0xFFFFu;
    }
    rl = total;
    if (lane == r - 1) rl_l = rl;
    __syncthreads();
  }
  if (!lower) {
    *bad = false;
    return 0;
  }
  // bought items, row by row (every wave by itself, 4 singles a lane; the
  // next row's positions on their way)
  const uint32_t pd = (m - le) + (rank - lt), single = m - 1 - pd;
  uint32_t len = 0, k = cap;
  bool ok = false, over = false;
  uint2 pos = reinterpret_cast<const uint2 *>(sm.spos[1])[lane];
#pragma unroll 1
  for (uint32_t r = 1; r <= L && k; ++r) {
    const uint2 p = pos;
    pos = reinterpret_cast<const uint2 *>(sm.spos[r < L ? r + 1 : L])[lane];
    if (k > static_cast<uint32_t>(__builtin_amdgcn_readlane(rl_l, r))) { over = true; break; }
    const uint32_t sg = static_cast<uint32_t>(__popcll(__ballot((p.x & 0xFFFF) < k)) + __popcll(__ballot((p.x >> 16) < k)) +
                                              __popcll(__ballot((p.y & 0xFFFF) < k)) + __popcll(__ballot((p.y >> 16) < k)));
    len += sg > single ? 1u : 0u;
    ok |= sg >= m;
    k = 2 * (k - sg);
  }
  *bad = over || !ok;
  return c && !*bad ? len : 0u;
}

// Code of one block per workgroup, a thread per symbol, leaf or node (the upper
// half of 512 ends after the lengths): its
// lengths (package-merge, or the supplied tree), then its layout.  A block
// with one symbol becomes a constant block; a present symbol without a code
// in the supplied tree is an argument error, and so are more symbols than
// codes of the limit's length; a block in error gets the constant mode
// (nothing to split) and sets *err.
// The code is canonical: with cnt(L) codes of length
// L and fc(L) the first of them, fc(L+1) = 2 (fc(L) + cnt(L)); a symbol's
// code is fc(len) plus its rank among the symbols of its length; the internal
// nodes at depth d are the prefixes [fc(d) + cnt(d), 2^d) numbered
// breadth-first, and child q of such a node is a leaf iff q < fc(d+1) +
// cnt(d+1).  With flat-subtree trees (shape 1, Sec. 2.2.3-2.2.4) the same
// closed form runs over the tree's items: the symbols of length L are cut by
// the binary digits of cnt(L), largest group first, a group of 2^D hanging at
// depth L - D; the items of a depth are ordered by D descending; a group of
// two or more symbols is a node (flat when D >= 2), numbered before the
// depth's internal nodes.  A node's counts are differences of the counts'
// prefix sums in leaf order at the ends of its leaf interval.
struct LayoutSmem {
  union {
  TreeSmem tree;
  struct {
  uint32_t wc[4][16];      // per wave: symbols of each length
  uint32_t cnt[18], ci[18], gn[18], fc[18], lvl[18], lb[18], kb[18];   // lb: leaves above depth d
  uint32_t pc[257];        // counts before each leaf
  uint16_t lo[256];
  uint32_t wsum[5][4];
  };
  };
  uint64_t present[4];     // per wave: its present symbols
};

// Sum of the values of the waves before this one, and of all, for the five
// scans of the layout.
__device__ __forceinline__ uint32_t waves_before(const uint32_t *w, uint32_t wave, uint32_t *all) {
  uint32_t b = 0, t = 0;
#pragma unroll
  for (uint32_t i = 0; i < 4; ++i) {
    const uint32_t x = w[i];
    b += i < wave ? x : 0u;
    t += x;
  }
  *all = t;
  return b;
}

// The end of a block's layout (one thread).  Without entropy-coded nodes its
// size is known here; a call of one block places it here too, what k_scan
// does for more.
__device__ void block_done(uint32_t ans_mode, uint32_t nb, BlockLay &L, uint8_t *H, uint32_t *err, Totals *tot,
                           const Result &res) {
  if (ans_mode == 0) {
    L.comp = L.hlen + L.raw_bytes;
    *reinterpret_cast<uint32_t *>(H) = L.comp;
  }
  if (nb != 1) return;
  L.ans0 = 0;
  if (ans_mode == 0) {
    L.out_off = stream_tables(1);
    L.img_off = L.out_off + L.hlen;
    tot->ans_words = 0;
    tot->out_bytes = L.out_off + ((static_cast<uint64_t>(L.comp) + 3) & ~3ull);
    finish(tot->out_bytes, err, res);
  } else {
    L.img_off = L.rbm_off = L.chunk0 = L.slot0 = 0;
    tot->img_bytes = img_area(L);
    tot->rbm_words = rbm_area(L);
    tot->chunks = L.n_chunks;
    tot->slot_bytes = L.slot_bytes;
    tot->ans_words = L.ans_words;
  }
}

template <uint32_t NT>
__global__ __launch_bounds__(NT) void k_code(
    const uint32_t *hist, uint32_t nb, uint64_t n, uint32_t bs, uint32_t max_len, pivco_tree tree,
    uint32_t use_tree, uint32_t ans_mode, uint32_t chunk_log2, uint32_t shape, const uint8_t *fse_dmax,
    EncBlock *eb, BlockLay *lay, RansNode *rnodes, uint8_t *hdr, uint32_t *err, Totals *tot, Result res) {
  __shared__ LayoutSmem sm;
  const uint32_t t = threadIdx.x, lane = __lane_id();
  const uint32_t wave = __builtin_amdgcn_readfirstlane(t >> 6);
  const uint32_t b = blockIdx.x;
  EncBlock &E = eb[b];
  BlockLay &Lb = lay[b];
  uint8_t *H = hdr + static_cast<uint64_t>(b) * kHdrStride;
  const uint64_t start = static_cast<uint64_t>(b) * bs;
  const uint32_t nblk = static_cast<uint32_t>(n - start < bs ? n - start : bs);
  const uint32_t cw = nblk <= 65535 ? 2u : 4u;
  const uint32_t c = wave < 4 ? hist[256ull * b + t] : 0u;   // the symbol's count
  // its length l, and the block's mode (0 coded, 1 | symbol << 8 constant)
  uint32_t mode = 0, l = 0;
  {
    const uint64_t bal = __ballot(c != 0);
    if (wave < 4) {
      if (lane == 0) sm.present[wave] = bal;
      sm.tree.cnt[t] = c;
    }
    __syncthreads();
    uint32_t m = 0, sym = 0;
#pragma unroll
    for (int w = 3; w >= 0; --w) {
      const uint64_t p = sm.present[w];
      m += static_cast<uint32_t>(__popcll(p));
      if (p) sym = 64 * w + static_cast<uint32_t>(__ffsll(static_cast<long long>(p))) - 1;
    }
    bool bad = false;
    if (use_tree) {
      l = tree.code_len[t & 255];
      bad = __syncthreads_or(c && l == 0);
      mode = bad ? 1u : 0u;
    } else if (m <= 1 || m > (1u << max_len)) {   // constant block, or no code of this length exists
      mode = 1u | (sym << 8);
      bad = m != 1;
    } else {
      l = nblk < (1u << 24) ? tree_lengths<NT, uint32_t>(sm.tree, m, max_len, &bad)
                            : tree_lengths<NT, uint64_t>(sm.tree, m, max_len, &bad);
      mode = bad ? 1u : 0u;
      __syncthreads();                       // the tables of the layout take the same memory
    }
    if (wave >= 4) return;                   // a barrier waits for the waves that are left
    if (bad && t == 0) atomicCAS(err, 0u, kErrArg);
  }
  if (t == 0) {
    E.in_off = start;
    E.n = nblk;
    Lb.n = nblk;
    *reinterpret_cast<uint32_t *>(H + 4) = nblk;
    H[8] = static_cast<uint8_t>(mode & 1);
    H[9] = static_cast<uint8_t>(mode >> 8);
    H[10] = static_cast<uint8_t>(cw);
    H[11] = 0;
  }
  if (mode & 1) {                        // constant block: its 12-byte header only
    if (t == 0) {
      E.I = 0;
      E.maxlen = 0;
      Lb.hlen = kBlockFixed;
      Lb.raw_bytes = Lb.ans_words = Lb.n_rnodes = Lb.n_chunks = 0;
      Lb.slot_bytes = 0;
      block_done(ans_mode, nb, Lb, H, err, tot, res);
    }
    return;
  }
  // the symbol's rank among the symbols of its length
  uint32_t rank = 0, wcl = 0;
#pragma unroll
  for (uint32_t L = 1; L <= 15; ++L) {
    const uint64_t mk = __ballot(l == L);
    const uint32_t before = __builtin_amdgcn_mbcnt_hi(static_cast<uint32_t>(mk >> 32),
                                                      __builtin_amdgcn_mbcnt_lo(static_cast<uint32_t>(mk), 0u));
    if (l == L) rank = before;
    if (lane == L) wcl = static_cast<uint32_t>(__popcll(mk));
  }
  if (lane < 16) sm.wc[wave][lane] = wcl;
  sm.pc[t] = 0;
  __syncthreads();
  // per depth, in lane d of every wave: symbols, items, group nodes, flat
  // nodes, leaves, first code, first node, leaves above
  uint32_t cnt_l = 0;
  if (lane < 16) cnt_l = sm.wc[0][lane] + sm.wc[1][lane] + sm.wc[2][lane] + sm.wc[3][lane];
  for (uint32_t w = 0; w < wave; ++w) rank += sm.wc[w][l & 15];
  uint32_t ci_l = cnt_l, gn_l = 0, nf_l = 0, nl_l = cnt_l;
  if (shape) {
    ci_l = nl_l = 0;
#pragma unroll
    for (uint32_t D = 0; D <= 8; ++D) {
      const uint32_t src = lane + D;
      const uint32_t cd = __shfl(cnt_l, static_cast<int>(src & 63), kWaveE);
      if (src <= 15 && ((cd >> D) & 1)) {
        ++ci_l;
        nl_l += 1u << D;
        gn_l += D >= 1 ? 1u : 0u;
        nf_l += D >= 2 ? 1u : 0u;
      }
    }
  }
  const uint64_t has_items = __ballot(lane <= 15 && ci_l != 0);
  const uint32_t maxitem = has_items ? 63u - static_cast<uint32_t>(__clzll(static_cast<long long>(has_items))) : 0u;
  uint32_t fc_l = 0, lvl_l = 0, fcd = 0, lvd = 0;
#pragma unroll
  for (uint32_t d = 0; d <= 16; ++d) {
    const uint32_t cd = __builtin_amdgcn_readlane(ci_l, d), gd = __builtin_amdgcn_readlane(gn_l, d);
    lvd += gd + (d < maxitem ? (1u << d) - fcd - cd : 0u);
    fcd = 2 * (fcd + cd);
    if (lane == d + 1) { fc_l = fcd; lvl_l = lvd; }
  }
  const uint32_t levels = maxitem + (__builtin_amdgcn_readlane(gn_l, maxitem) ? 1u : 0u);
  const uint32_t I = __builtin_amdgcn_readlane(lvl_l, levels);
  const uint32_t lsum = wave_incl_scan(lane < 16 ? nl_l : 0u);
  const uint32_t nleaf = __builtin_amdgcn_readlane(lsum, 63);
  // canonical: internal nodes only, p - fc - ci of the level; flat-subtree:
  // every prefix of the level from its first item on
  const uint32_t single = shape && lane < 16 ? ci_l - gn_l : 0u;
  const uint32_t kb_l = shape ? lvl_l - fc_l + wave_incl_scan(single) - single : lvl_l - fc_l - ci_l;
  if (wave == 0) {
    if (lane < 18) {
      sm.kb[lane] = kb_l;
      sm.cnt[lane] = cnt_l; sm.ci[lane] = lane < 16 ? ci_l : 0u; sm.gn[lane] = gn_l;
      sm.fc[lane] = fc_l; sm.lvl[lane] = lvl_l; sm.lb[lane] = lsum - (lane < 16 ? nl_l : 0u);
      E.lvl[lane] = lvl_l;
    }
    if (lane < 16) {
      E.kbase[lane] = static_cast<int32_t>(kb_l);
      E.nfl[lane] = static_cast<uint8_t>(nf_l);
    }
    if (lane == 0) { E.maxlen = levels; E.I = I; E.nleaf = nleaf; }
  }
  __syncthreads();
  // codes, and the leaves in code order
  uint32_t pay = 0;
  if (l) {
    uint32_t code, leaf;
    if (shape == 0) {
      code = sm.fc[l] + rank;
      leaf = sm.lb[l] + rank;
    } else {
      const uint32_t cn = sm.cnt[l];     // the symbol's group: binary digits of cnt(l), largest first
      uint32_t D = 0, first = 0;
      for (uint32_t e = 9; e-- > 0;) {
        if (!((cn >> e) & 1)) continue;
        if (rank < first + (1u << e)) { D = e; break; }
        first += 1u << e;
      }
      const uint32_t m = l - D;
      uint32_t idx = 0, lv = 0;          // items of depth m with a larger D, and their leaves
      for (uint32_t e = D + 1; e <= 8; ++e)
        if (m + e <= 15 && ((sm.cnt[m + e] >> e) & 1)) { ++idx; lv += 1u << e; }
      code = ((sm.fc[m] + idx) << D) | (rank - first);
      leaf = sm.lb[m] + lv + (rank - first);
    }
    pay = code << (16 - l);
    sm.pc[leaf] = c;
    E.leaf[t] = static_cast<uint8_t>(leaf);
  } else {
    E.leaf[t] = 255;
  }
  E.pay[t] = static_cast<uint16_t>(pay);
  __syncthreads();
  {
    const uint32_t own = sm.pc[t], inc = wave_incl_scan(own);
    if (lane == kWaveE - 1) sm.wsum[0][wave] = inc;
    __syncthreads();
    uint32_t all;
    const uint32_t ex = waves_before(sm.wsum[0], wave, &all) + inc - own;
    sm.pc[t] = ex;
    if (t == 255) sm.pc[256] = all;
  }
  // node t: depth, children, first leaf
  uint32_t d = 0, fd = 0, cc = 0, lo = 0, hi = 0, slot = 0;
  bool group = false;
  const bool node = t < I;
  if (node) {
    for (uint32_t j = 1; j < levels; ++j) d += t >= sm.lvl[j] ? 1u : 0u;
    const uint32_t r = t - sm.lvl[d];
    if (r < sm.gn[d]) {                  // group r of depth d (shape 1)
      uint32_t D = 0, left = r, lv = 0;
      for (uint32_t e = 8; e >= 1; --e)
        if (d + e <= 15 && ((sm.cnt[d + e] >> e) & 1)) {
          if (left == 0) { D = e; break; }
          --left;
          lv += 1u << e;
        }
      group = true;
      slot = sm.fc[d] + r + sm.kb[d];
      lo = sm.lb[d] + lv;
      hi = lo + (1u << D);
      cc = 0x80008000u;
      fd = D >= 2 ? D : 0u;
    } else {
      const uint32_t p = sm.fc[d] + sm.ci[d] + (r - sm.gn[d]);
      const uint32_t d1 = d + 1;
      slot = p + sm.kb[d];
      for (int bb = 0; bb < 2; ++bb) {
        const uint32_t q = 2 * p + bb;
        const uint32_t rq = q - sm.fc[d1];
        const uint32_t ch = rq < sm.gn[d1] ? sm.lvl[d1] + rq
                            : rq < sm.ci[d1] ? 0x8000u
                                             : sm.lvl[d1] + sm.gn[d1] + (q - sm.fc[d1] - sm.ci[d1]);
        cc |= ch << (16 * bb);
      }
      // the first leaf: the item that the leftmost path under p ends in
      for (uint32_t e = d1; e <= 16; ++e) {
        const uint32_t x = (p << (e - d)) - sm.fc[e];
        if (x >= sm.ci[e]) continue;
        lo = sm.lb[e];
        if (shape == 0) {
          lo += x;
        } else {
          uint32_t left = x;
          for (uint32_t g = 8; left; --g)
            if (e + g <= 15 && ((sm.cnt[e + g] >> g) & 1)) { lo += 1u << g; --left; }
        }
        break;
      }
    }
    sm.lo[t] = static_cast<uint16_t>(lo);
  }
  __syncthreads();
  uint32_t nv = 0, nr = 0, mk = 0, kd = 0;
  if (node) {
    if (!group) hi = t + 1 < sm.lvl[d + 1] ? sm.lo[t + 1] : nleaf;
    const uint32_t c1 = cc >> 16;
    const uint32_t mid = fd ? hi : (c1 & 0x8000) ? hi - 1 : sm.lo[c1];
    nv = sm.pc[hi] - sm.pc[lo];
    nr = sm.pc[hi] - sm.pc[mid];
    *reinterpret_cast<uint16_t *>(E.child[t]) = static_cast<uint16_t>(((cc & 0x8000) ? 255u : cc & 255) |
                                                                      ((c1 & 0x8000) ? 255u : c1) << 8);
    E.lo[t] = static_cast<uint8_t>(lo);
    E.mid1[t] = static_cast<uint8_t>(mid - 1);
    E.hi1[t] = static_cast<uint8_t>(hi - 1);
    E.depth[t] = static_cast<uint8_t>(d);
    E.fd[t] = static_cast<uint8_t>(fd);
    E.slot[t] = static_cast<uint8_t>(slot - t);
    if (!fd) {
      if (ans_mode == 3) mk = fse_marker(nv, nr, d, fse_dmax);
      kd = (ans_mode == 3 ? mk != 0 : select_ans(ans_mode, nv, nr)) ? 1u : 0u;
    }
  }
  // sizes of the node's parts and their prefixes
  const uint32_t C = 1u << chunk_log2;
  const uint32_t nch = kd ? (nv + C - 1) >> chunk_log2 : 0u;
  const uint32_t rem = nv - (nch ? (nch - 1) * C : 0u);
  const uint64_t bits = static_cast<uint64_t>(nv) * (fd ? fd : 1u);
  const uint32_t part[5] = {kd || !node ? 0u : static_cast<uint32_t>((bits + 7) / 8), kd ? (nv + 31) / 32 : 0u, kd, nch,
                            nch ? ((nch - 1) * slot_size(C) + slot_size(rem)) / 16 : 0u};   // slots in 16-byte units
  uint32_t ex[5], all[5];
#pragma unroll
  for (int q = 0; q < 5; ++q) {
    ex[q] = wave_incl_scan(part[q]);
    if (lane == kWaveE - 1) sm.wsum[q][wave] = ex[q];
  }
  __syncthreads();
#pragma unroll
  for (int q = 0; q < 5; ++q) ex[q] += waves_before(sm.wsum[q], wave, &all[q]) - part[q];
  if (node) E.bit[t] = kd ? ex[1] : ex[0];
  if (kd) {
    RansNode r;
    r.rword = ex[1];
    r.nv = nv;
    r.p1q = ans_mode == 3 ? mk : p1q_of(nv, nr);
    r.ch0 = ex[3];
    r.sl0 = 16ull * ex[4];
    rnodes[255ull * b + ex[2]] = r;
  }
  // header: code lengths (two nibbles a byte, symbol 2j low), kind bits, counts of 1 bits
  const uint32_t kb = (I + 7) / 8;
  const uint32_t l_next = __shfl_down(l, 1, kWaveE);
  if ((t & 1) == 0) H[12 + t / 2] = static_cast<uint8_t>(l | (l_next << 4));
  const uint64_t km = __ballot(kd);
  if (lane < 2) E.kind[2 * wave + lane] = static_cast<uint32_t>(km >> (32 * lane));
  if (lane < 8 && 8 * wave + lane < kb) H[140 + 8 * wave + lane] = static_cast<uint8_t>(km >> (8 * lane));
  if (node) {
    uint8_t *q = H + 140 + kb + cw * t;
    q[0] = static_cast<uint8_t>(nr);
    q[1] = static_cast<uint8_t>(nr >> 8);
    if (cw == 4) { q[2] = static_cast<uint8_t>(nr >> 16); q[3] = static_cast<uint8_t>(nr >> 24); }
  }
  if (t == 0) {
    Lb.hlen = 140 + kb + cw * I;
    Lb.raw_bytes = all[0];
    Lb.ans_words = all[1];
    Lb.n_rnodes = all[2];
    Lb.n_chunks = all[3];
    Lb.slot_bytes = 16ull * all[4];
    block_done(ans_mode, nb, Lb, H, err, tot, res);
  }
}

// Exclusive scans over the blocks (one workgroup, a block per thread): with
// entropy-coded nodes image bytes, rANS bitmap words, chunk jobs, slot bytes
// and scratch words, and their totals; without them the blocks' places in the
// stream, and the call's result.
__global__ __launch_bounds__(kScanNT) void k_scan(BlockLay *lay, uint32_t nb, uint32_t ans_mode, Totals *tot,
                                                  uint32_t *err, Result res) {
  __shared__ uint64_t part[kScanNT / kWaveE];
  const uint32_t tid = threadIdx.x;
  uint64_t run[5] = {ans_mode ? 0ull : stream_tables(nb), 0, 0, 0, 0};
  for (uint64_t b0 = 0; b0 < nb; b0 += kScanNT) {
    const uint64_t b = b0 + tid;
    uint64_t v[5] = {0, 0, 0, 0, 0}, x[5], all[5];
    if (b < nb) {
      const BlockLay &L = lay[b];
      if (ans_mode) {
        v[0] = img_area(L);
        v[1] = rbm_area(L);
        v[2] = L.n_chunks;
        v[3] = L.slot_bytes;
        v[4] = L.ans_words;
      } else {
        v[0] = (static_cast<uint64_t>(L.comp) + 3) & ~3ull;
      }
    }
    for (int q = 0; q < 5; ++q) {
      if (q && !ans_mode) break;
      x[q] = run[q] + block_excl_scan(v[q], part, &all[q]);
      run[q] += all[q];
    }
    if (b < nb) {
      BlockLay &L = lay[b];
      if (ans_mode) {
        L.img_off = x[0];
        L.rbm_off = x[1];
        L.chunk0 = x[2];
        L.slot0 = x[3];
        L.ans0 = x[4];
      } else {
        L.out_off = x[0];
        L.img_off = x[0] + L.hlen;
        L.ans0 = 0;
      }
    }
  }
  if (tid != 0) return;
  if (ans_mode) {
    tot->img_bytes = run[0];
    tot->rbm_words = run[1];
    tot->chunks = run[2];
    tot->slot_bytes = run[3];
    tot->ans_words = run[4];
  } else {
    tot->ans_words = 0;
    tot->out_bytes = run[0];
    finish(run[0], err, res);
  }
}

// LDS-only workgroup barrier (the split kernel's waves share nothing else).
__device__ __forceinline__ void lds_sync() {
  __builtin_amdgcn_fence(__ATOMIC_RELEASE, "workgroup", "local");
  __builtin_amdgcn_s_barrier();
  __builtin_amdgcn_fence(__ATOMIC_ACQUIRE, "workgroup", "local");
}

static_assert(kMaxLenGpu <= 12, "code bits of a symbol");
// The chunk jobs of a block's rANS nodes, a node per thread of nt.
__device__ void chunk_jobs(const BlockLay &L, const RansNode *rnodes, uint32_t b, uint32_t chunk_log2, uint32_t nt,
                           RansJob *jobs) {
  const uint32_t C = 1u << chunk_log2;
  for (uint32_t r = threadIdx.x; r < L.n_rnodes; r += nt) {
    const RansNode rn = rnodes[r];
    uint32_t k = 0;
    for (uint64_t st = 0; st < rn.nv; st += C, ++k) {
      RansJob j;
      j.bmp_word = L.rbm_off + rn.rword + st / 32;
      j.slot = L.slot0 + rn.sl0 + static_cast<uint64_t>(k) * slot_size(C);
      j.nbits = rn.nv - st < C ? static_cast<uint32_t>(rn.nv - st) : C;
      j.p1q = rn.p1q;
      j.block = b;
      j.rnode = r;
      j.first = st == 0;
      j.dst = 0;
      jobs[L.chunk0 + rn.ch0 + k] = j;
    }
  }
}

constexpr uint32_t kEndsHere = 0x7F00;   // SplitSmem::K of a leaf: past every place (in bytes)

template <int NT, uint32_t S>
struct SplitSmem {
  union {
    uint32_t bits[13 * S / 32 + 2 * 16 + 4];   // every level's bits, then the flat nodes' fields
    struct {                           // before the levels only
      uint32_t P[257], C[257];         // symbols of the slice / of earlier slices before each leaf
      uint32_t T[257], O[257];         // symbols / 1 bits of the nodes before each node
    };
  };
  // a level's codes, in its nodes' order (groups of 4 chunks read past its
  // end; not first, as a place less the chunks done may be below 0)
  uint16_t buf[S + 64 * 4];
  int16_t K[2 * 272];                  // node in slot i: [2i] where its 0 symbols go, [2i + 1] its 1 symbols, in bytes (see k_split)
  uint32_t F[272];                     // flat node, by slot: where its fields go | D << 24
  uint32_t wx[257];                    // output words of the nodes before each node
  uint32_t src[256], len[256];         // node's first bit in `bits`; bits | rANS << 31
  uint64_t q[256];                     // node's first bit in its area
  uint16_t pay[256];
  uint32_t lvl[18], fbits;             // levels' first nodes; flat fields' bits
  uint32_t wsum[2][NT / kWaveE];
  uint32_t part[4][NT / kWaveE];
};

// 32 bits from bit x of an LDS word array.
__device__ __forceinline__ uint32_t bits32(const uint32_t *w, uint32_t x) {
  return __builtin_amdgcn_alignbit(w[(x >> 5) + 1], w[x >> 5], x & 31);
}

// One workgroup per slice of kSlice symbols of a block (slice k of block b is
// workgroup b * spb + k).
//   Nodes: the slice's counts (from the prefix histograms) summed in leaf
// order give every node's symbols and 1 bits in the slice, and the symbols
// of earlier slices where its bits go on; scans over the nodes place each
// node in its level.
//   Levels: a level's symbols lie in one array, nodes in breadth-first order
// and stream order inside a node, so each wave takes an equal share of it in
// 64-symbol chunks whatever the nodes' sizes.  A chunk's bits are one ballot,
// stored as 64 bits of the level's bit array; R(p), the 1 bits of the level
// before position p, is the ballots' running count, and a symbol at p goes to
// p - R(p) + K (0 bit) or R(p) + K (1 bit): K, by the code's bits so far, holds the child's
// place less the node's own terms, and for a leaf (the symbol ends there) a
// value past every place.  The symbols of a flat node end in it and store their D-bit
// index at D times their place.
//   Output: the nodes' bits are copied out of the level arrays word by word,
// at the bit where the node's earlier slices end.  A raw node goes to its
// byte offset in the block's raw image (the stream layout), a rANS node to its
// word among the block's rANS bitmap words; without entropy-coded nodes
// (direct: the stream's totals) img is the stream itself, where the blocks'
// places are known and k_head has zeroed the bodies.  A word that this slice
// does not fill is ORed into zeroed memory, the others are stored.
//   The first slice's workgroup also lists the block's chunk jobs.
// Bound by vector instructions (four fifths of the issue slots), about 21 per 64
// symbols and level (522M of the 634M of 256 MiB Zipf(1.1)), and by the latency of
// the small levels (two barriers each).  Symbols that end are stored to one unused
// place instead of being masked off, a place is one shift and add from the rank,
// and waves take whole groups of 4 chunks: 690M -> 634M, 1.39 -> 1.31 ms.  256 MiB
// Zipf(1.1) in 64 KiB blocks: 1.31 ms where one wave per node (the root's 4096
// symbols on one wave of four) took 4.15 ms; one 64 KiB block: 18 us, was 86.  LDS
// holds one
// level buffer (a level is in registers before it moves) and no more tables
// than the levels need, for 6 workgroups of 256 threads on a CU: with two
// buffers and the tables beside them (4 workgroups) and the block's tables
// read in a chain it took 2.7 ms.
template <int NT, uint32_t kSlice, bool FLAT>
__global__ __launch_bounds__(NT) void k_split(const uint8_t *in, const EncBlock *blocks,
                                              const BlockLay *lay, uint32_t nblocks, uint32_t spb,
                                              const uint32_t *pre, const uint32_t *hist, uint32_t *img,
                                              uint32_t *rbm, const Totals *direct, uint64_t out_cap,
                                              const RansNode *rnodes, uint32_t chunk_log2, RansJob *jobs) {
  constexpr int kSplitNT = NT, kSplitNW = NT / kWaveE;
  constexpr uint32_t kPer = kSlice / NT;     // symbols of a thread, and 64-symbol chunks of a wave, at most
  constexpr uint32_t kSplitCh = kPer;
  static_assert(kSlice <= 8192 && kPer % 4 == 0 && kPer <= 16, "places and leaf marks in 16 signed bits");
  __shared__ __attribute__((aligned(16))) SplitSmem<NT, kSlice> sm;
  const uint32_t tid = threadIdx.x, lane = __lane_id();
  const uint32_t wave = __builtin_amdgcn_readfirstlane(tid >> 6);
  const uint32_t b = blockIdx.x / spb, slice = blockIdx.x % spb;
  if (b >= nblocks || (direct && direct->out_bytes > out_cap)) return;
  if (jobs && slice == 0) chunk_jobs(lay[b], rnodes + 255ull * b, b, chunk_log2, NT, jobs);
  const EncBlock &B = blocks[b];
  const uint32_t I = B.I, n = B.n, s_lo = slice * kSlice;
  if (I == 0 || s_lo >= n) return;
  const uint32_t S = n - s_lo < kSlice ? n - s_lo : kSlice;
  const uint32_t levels = B.maxlen;
  // everything the slice needs from memory, in one round trip: its symbols
  // (kPer consecutive ones a thread, no alignment), the symbol's and the node's
  // row of the block's tables, the levels' values (one level a lane)
  const uint8_t *src = in + B.in_off + s_lo;
  uint32_t sy[kPer / 4] = {};
  if (kPer * (tid + 1) <= S) {
    __builtin_memcpy(sy, src + kPer * tid, kPer);
  } else {
#pragma unroll
    for (uint32_t e = 0; e < kPer; ++e)
      if (kPer * tid + e < S) sy[e >> 2] |= static_cast<uint32_t>(src[kPer * tid + e]) << (8 * (e & 3));
  }
  uint32_t cnt = 0, bef = 0, leaf = 0, lo = 0, mid = 0, hi = 0, cc = 0, d = 0, slot = 0, fd = 0, nbit = 0, pay = 0;
  bool rans = false;
  const bool first256 = NT == 256 || tid < 256;
  if (first256) {
    const uint32_t *row = pre + static_cast<uint64_t>(blockIdx.x) * 256 + tid;
    bef = slice ? row[0] : 0u;
    cnt = slice + 1 < spb ? row[256] : hist[256ull * b + tid];
    leaf = B.leaf[tid];
    pay = B.pay[tid];
    lo = B.lo[tid];
    mid = B.mid1[tid] + 1u;
    hi = B.hi1[tid] + 1u;
    cc = *reinterpret_cast<const uint16_t *>(B.child[tid]);
    d = B.depth[tid];
    slot = B.slot[tid] + tid;
    if (FLAT) fd = B.fd[tid];
    nbit = B.bit[tid];
    rans = (B.kind[tid >> 5] >> (tid & 31)) & 1;
  }
  const uint64_t img_off = lay[b].img_off, rbm_off = lay[b].rbm_off;
  const uint32_t lvl_l = B.lvl[lane < 18 ? lane : 0u], kb_l = static_cast<uint32_t>(B.kbase[lane & 15]);
  const uint32_t nfl_l = FLAT ? B.nfl[lane & 15] : 0u;
  if (first256) {
    cnt -= bef;
    sm.pay[tid] = static_cast<uint16_t>(pay);
    sm.P[leaf] = cnt;
    sm.C[leaf] = bef;
  }
  if (tid < 18) sm.lvl[tid] = lvl_l;
  lds_sync();
  // counts in leaf order become prefix sums (entries past the last leaf are
  // not written above and change no prefix that is read)
  if (wave < 4) {
    cnt = sm.P[tid & 255];
    bef = sm.C[tid & 255];
    const uint32_t ic = wave_incl_scan(cnt), ib = wave_incl_scan(bef);
    cnt = ic - cnt;
    bef = ib - bef;
    if (lane == kWaveE - 1) { sm.part[0][wave] = ic; sm.part[1][wave] = ib; }
  }
  // the root level: every symbol's code
  {
    uint32_t w[kPer / 2];
#pragma unroll
    for (uint32_t e = 0; e < kPer / 2; ++e) {
      const uint32_t x = (sy[e >> 1] >> (16 * (e & 1))) & 255, y = (sy[e >> 1] >> (16 * (e & 1) + 8)) & 255;
      w[e] = sm.pay[x] | (static_cast<uint32_t>(sm.pay[y]) << 16);
    }
    uint2 *dst = reinterpret_cast<uint2 *>(sm.buf) + kPer / 4 * tid;
#pragma unroll
    for (uint32_t e = 0; e < kPer / 4; ++e) dst[e] = make_uint2(w[2 * e], w[2 * e + 1]);
  }
  lds_sync();
  if (wave < 4) {
    uint32_t ac, ab;
    cnt += waves_before(sm.part[0], wave, &ac);
    bef += waves_before(sm.part[1], wave, &ab);
    sm.P[tid] = cnt;
    sm.C[tid] = bef;
    if (tid == 0) { sm.P[256] = ac; sm.C[256] = ab; }
  }
  lds_sync();
  // node tid
  const bool node = tid < I;
  uint32_t tv = 0, ones = 0, nw = 0, fx = 0;
  if (wave < 4) {
    uint32_t fb = 0;
    if (node) {
      tv = sm.P[hi] - sm.P[lo];
      ones = sm.P[hi] - sm.P[mid];
      const uint32_t cur = sm.C[hi] - sm.C[lo], D = FLAT && fd ? fd : 1u;
      const uint64_t q = (rans ? 32 * (rbm_off + nbit) : 8 * (img_off + nbit)) + static_cast<uint64_t>(D) * cur;
      const uint32_t len = D * tv;
      nw = len ? (static_cast<uint32_t>(q & 31) + len + 31) / 32 : 0u;
      fb = FLAT && fd ? len : 0u;
      sm.q[tid] = q;
      sm.len[tid] = len | (rans ? 0x80000000u : 0u);
    }
    const uint32_t it = wave_incl_scan(tv), io = wave_incl_scan(ones), iw = wave_incl_scan(nw);
    const uint32_t jf = FLAT ? wave_incl_scan(fb) : 0u;
    if (lane == kWaveE - 1) {
      sm.part[0][wave] = it; sm.part[1][wave] = io; sm.part[2][wave] = iw; sm.part[3][wave] = jf;
    }
    tv = it - tv;
    ones = io - ones;
    nw = iw - nw;
    fx = jf - fb;
  }
  lds_sync();
  if (wave < 4) {
    uint32_t at, ao, aw, af = 0;
    tv += waves_before(sm.part[0], wave, &at);        // from here on the sums before this node
    ones += waves_before(sm.part[1], wave, &ao);
    nw += waves_before(sm.part[2], wave, &aw);
    if (FLAT) fx += waves_before(sm.part[3], wave, &af);
    sm.T[tid] = tv;
    sm.O[tid] = ones;
    sm.wx[tid] = nw;
    if (tid == 0) { sm.T[256] = at; sm.O[256] = ao; sm.wx[256] = aw; sm.fbits = af; }
  }
  lds_sync();
  // per level, in lane d of every wave: symbols, those in flat nodes, first
  // 64-bit word of its bits
  uint32_t ln_l = 0, lf_l = 0;
  if (lane < levels) {
    const uint32_t t0 = sm.T[lvl_l];
    ln_l = sm.T[sm.lvl[lane + 1]] - t0;
    if (FLAT) lf_l = sm.T[lvl_l + nfl_l] - t0;
  }
  const uint32_t w64 = (ln_l + 63) / 64, lw_i = wave_incl_scan(w64), lw_l = lw_i - w64;
  const uint32_t all64 = __builtin_amdgcn_readlane(lw_i, 63), fbits = FLAT ? sm.fbits : 0u;
  const uint32_t lw_d = __shfl(lw_l, static_cast<int>(d), kWaveE);   // every lane takes part
  if (node) {
    const uint32_t l0 = sm.lvl[d], l1 = sm.lvl[d + 1];
    const uint32_t seg = tv - sm.T[l0], rs = ones - sm.O[l0], t1 = sm.T[l1];
    const uint32_t c0 = cc & 255, c1 = cc >> 8;
    const uint32_t k0 = c0 == 255 ? kEndsHere : 2 * (sm.T[c0] - t1 - seg + rs) & 0xFFFF;
    const uint32_t k1 = c1 == 255 ? kEndsHere : 2 * (sm.T[c1] - t1 - rs) & 0xFFFF;
    reinterpret_cast<uint32_t *>(sm.K)[slot] = k0 | (k1 << 16);
    const uint32_t sb = FLAT && fd ? 64 * all64 + fx : 64 * lw_d + seg;
    if (FLAT) sm.F[slot] = ((sb - fd * seg) & 0xFFFFFF) | (fd << 24);   // bit sb + D (p - seg)
    sm.src[tid] = sb;
  }
  lds_sync();
  // the flat fields are ORed in, from the second half of the root level on
  if (FLAT)
    for (uint32_t i = tid; i < (fbits + 31) / 32; i += kSplitNT) sm.bits[2 * all64 + i] = 0;
  uint32_t next = __builtin_amdgcn_readlane(ln_l, 0);
  for (uint32_t lev = 0; lev < levels; ++lev) {
    const uint32_t ln = next;
    if (ln == 0) break;
    const uint32_t lf = FLAT ? __builtin_amdgcn_readlane(lf_l, lev) : 0u;
    next = __builtin_amdgcn_readlane(ln_l, lev + 1);
    const uint32_t nch = (ln + 63) / 64, least = (nch + kSplitNW - 1) / kSplitNW;
    const uint32_t per = NT > 512 ? least : (least + 3) & ~3u;   // whole groups where several workgroups share a CU
    const uint32_t ch0 = wave * per, ch1 = ch0 + per < nch ? ch0 + per : nch;
    uint16_t *buf = sm.buf;              // every symbol is in registers before any moves
    uint2 *lbits = reinterpret_cast<uint2 *>(sm.bits) + __builtin_amdgcn_readlane(lw_l, lev);
    const uint32_t lim = 64 * ch1 < ln ? 64 * ch1 : ln;   // this wave's positions end here
    const uint32_t p0 = 64 * ch0 + lane;
    const uint32_t mask = 0x8000u >> lev;    // the level's bit (the ballots are made twice: kept, they spill)
    uint32_t pl[kSplitCh], run = 0;
    // groups of 4 chunks; a group inside the wave's share (and past the
    // level's flat nodes) needs no test per symbol
#pragma unroll
    for (uint32_t g = 0; g < kSplitCh; g += 4) {
      if (ch0 + g >= ch1) break;
      if (64 * (ch0 + g + 4) <= lim && (!FLAT || 64 * (ch0 + g) >= lf)) {
#pragma unroll
        for (uint32_t i = g; i < g + 4; ++i) pl[i] = buf[p0 + 64 * i];
        uint64_t m[4];
#pragma unroll
        for (uint32_t i = 0; i < 4; ++i) m[i] = __ballot(pl[g + i] & mask);
        if (lane == 0) {
#pragma unroll
          for (uint32_t i = 0; i < 4; ++i)
            lbits[ch0 + g + i] = make_uint2(static_cast<uint32_t>(m[i]), static_cast<uint32_t>(m[i] >> 32));
        }
#pragma unroll
        for (uint32_t i = 0; i < 4; ++i) run += static_cast<uint32_t>(__popcll(m[i]));
      } else {
#pragma unroll
        for (uint32_t i = g; i < g + 4; ++i) {
          if (ch0 + i >= ch1) break;
          const uint32_t p = p0 + 64 * i;
          pl[i] = buf[p];
          const uint64_t m = __ballot((pl[i] & mask) && p < lim && (!FLAT || p >= lf));
          if (lane == 0) lbits[ch0 + i] = make_uint2(static_cast<uint32_t>(m), static_cast<uint32_t>(m >> 32));
          run += static_cast<uint32_t>(__popcll(m));
        }
      }
    }
    if (next == 0 && lf == 0) break;         // every symbol ends here
    if (lane == 0) sm.wsum[lev & 1][wave] = run;
    lds_sync();
    if (ch0 < ch1) {
      uint32_t R = 0;
      if (kSplitNW <= 4) {
#pragma unroll
        for (uint32_t w = 0; w < kSplitNW; ++w) R += w < wave ? sm.wsum[lev & 1][w] : 0u;
      } else {
        R = __builtin_amdgcn_readlane(wave_incl_scan(lane < wave ? sm.wsum[lev & 1][lane & (kSplitNW - 1)] : 0u), 63);
      }
      // from here on R and a symbol's place are 32 less per chunk done: the
      // constant goes into the store's offset, also for p - R
      char *to = reinterpret_cast<char *>(buf);
      const int32_t kbase = static_cast<int32_t>(__builtin_amdgcn_readlane(kb_l, lev));
      const int16_t *Kl = sm.K + 2 * kbase;    // by the code's first lev + 1 bits
#pragma unroll
      for (uint32_t g = 0; g < kSplitCh; g += 4) {
        if (ch0 + g >= ch1) break;
        if (64 * (ch0 + g + 4) <= lim && (!FLAT || 64 * (ch0 + g) >= lf)) {
          int32_t k[4];
#pragma unroll
          for (uint32_t i = 0; i < 4; ++i) k[i] = Kl[pl[g + i] >> (15 - lev)];
#pragma unroll
          for (uint32_t i = 0; i < 4; ++i) {
            const bool bit = pl[g + i] & mask;
            const uint64_t mm = __ballot(bit);
            const uint32_t r = __builtin_amdgcn_mbcnt_hi(static_cast<uint32_t>(mm >> 32),
                                                         __builtin_amdgcn_mbcnt_lo(static_cast<uint32_t>(mm), R));
            R += static_cast<uint32_t>(__popcll(mm)) - 32u;
            const int32_t at = static_cast<int32_t>((bit ? r : p0 - r) << 1) + k[i];
            const int32_t off = 64 * static_cast<int32_t>(g + i), unused = 2 * (kSlice + 64) - off;
            *reinterpret_cast<uint16_t *>(to + (at < unused ? at : unused) + off) = static_cast<uint16_t>(pl[g + i]);
          }
        } else {
#pragma unroll
          for (uint32_t i = 0; i < 4; ++i) {
            if (ch0 + g + i >= ch1) break;
            const uint32_t p = p0 + 64 * (g + i), c = pl[g + i];
            const uint32_t v = p < lim ? (c >> (16 - lev)) + kbase : 0u;
            const int32_t k = sm.K[2 * v + ((c >> (15 - lev)) & 1)];
            const bool bit = (c & mask) && p < lim && (!FLAT || p >= lf);
            const uint64_t mm = __ballot(bit);
            const uint32_t r = __builtin_amdgcn_mbcnt_hi(static_cast<uint32_t>(mm >> 32),
                                                         __builtin_amdgcn_mbcnt_lo(static_cast<uint32_t>(mm), R));
            R += static_cast<uint32_t>(__popcll(mm)) - 32u;
            if (p >= lim) continue;
            if (FLAT && p < lf) {              // D-bit field: the code's last D bits
              const uint32_t F = sm.F[v], D = F >> 24, x = (F + D * p) & 0xFFFFFF;
              const uint32_t f = ((c << lev) & 0xFFFF) >> (16 - D);
              atomicOr(&sm.bits[x >> 5], f << (x & 31));
              if ((x & 31) + D > 32) atomicOr(&sm.bits[(x >> 5) + 1], f >> (32 - (x & 31)));
            } else {
              const uint32_t at = ((bit ? r : p0 - r) << 1) + k + 64 * (g + i);
              if (at < 2 * kSlice) *reinterpret_cast<uint16_t *>(to + at) = static_cast<uint16_t>(c);
            }
          }
        }
      }
    }
    lds_sync();
  }
  lds_sync();
  // output words
  const uint32_t words = sm.wx[256];
  for (uint32_t j = tid; j < words; j += kSplitNT) {
    uint32_t v = 0;                          // the last node whose words start at or before j
#pragma unroll
    for (uint32_t st = 128; st; st >>= 1) v += sm.wx[v + st] <= j ? st : 0u;
    const uint32_t k = j - sm.wx[v], lr = sm.len[v], len = lr & 0x7FFFFFFF;
    const uint64_t q = sm.q[v];
    const uint32_t sft = static_cast<uint32_t>(q & 31);
    uint32_t w = k ? bits32(sm.bits, sm.src[v] + 32 * k - sft) : bits32(sm.bits, sm.src[v]) << sft;
    const uint32_t end = sft + len - 32 * k;
    if (end < 32) w &= (1u << end) - 1;
    uint32_t *dst = ((lr >> 31) ? rbm : img) + (q >> 5) + k;
    if (end < 32 || (k == 0 && sft)) {
      if (w) atomicOr(dst, w);
    } else {
      *dst = w;
    }
  }
}

// x / f and x % f of the rANS step, folded into its new state: q * 4096 + r +
// add, for x < f * 2^20 and rcp = floor(2^32 / f) (2^32 - 1 for f = 1).  The
// high product is the quotient or one less, so one correction serves.
__device__ __forceinline__ uint32_t rans_next(uint32_t x, uint32_t f, uint32_t rcp, uint32_t add) {
  const uint32_t q = __umulhi(x, rcp), r = x - __umul24(q, f);
  return q * kRansM + r + add + (r >= f ? kRansM - f : 0u);
}

// One wave per chunk (persistent over the job list): encode steps k = K-1 ..
// 0; within a step the lanes push their renormalisation words in the order
// lane 31 .. 0, the reverse of the decoder's read order, so the decoder reads
// the pushed words backwards.  A step is a chain of dependent operations that
// sets the kernel's time, so nothing in it waits for memory (the words of 32
// steps sit in the lanes), the division is a product with the reciprocal, and
// 32 full steps are unrolled, which takes all that does not depend on the
// state off the chain: a chunk of 2^16 bits 384 -> 172 us.
__global__ __launch_bounds__(256) void k_rans_enc(const RansJob *jobs, const Totals *tot,
                                                  const uint32_t *bmp, uint8_t *slots,
                                                  uint32_t *sizes) {
  const uint32_t lane = __lane_id();
  const uint64_t njobs = tot->chunks;
  const uint64_t nwaves = static_cast<uint64_t>(gridDim.x) * (256 / kWaveE);
  for (uint64_t j = blockIdx.x * (256 / kWaveE) + (threadIdx.x >> 6); j < njobs; j += nwaves) {
    const RansJob J = jobs[j];
    const uint32_t f0 = kRansM - J.p1q, f1 = J.p1q;    // both in [1, 4095]
    const uint32_t rcp0 = f0 > 1 ? static_cast<uint32_t>((1ull << 32) / f0) : 0xFFFFFFFFu;
    const uint32_t rcp1 = f1 > 1 ? static_cast<uint32_t>((1ull << 32) / f1) : 0xFFFFFFFFu;
    const uint32_t K = (J.nbits + 31) / 32;
    uint8_t *slot = slots + J.slot;
    uint16_t *words = reinterpret_cast<uint16_t *>(slot + kChunkHdr);
    const uint32_t *bits = bmp + J.bmp_word;
    uint32_t x = kRansL;
    uint32_t pos = 0;
    if (lane < kRansLanes) {
      const uint32_t gt = lane < 31 ? ~((2u << lane) - 1) : 0u;   // lanes above this one
      auto step = [&](uint32_t w, bool act) {
        const bool bit = (w >> lane) & 1;
        const uint32_t f = bit ? f1 : f0;
        const bool need = act && x >= (f << 20);
        const uint32_t m = static_cast<uint32_t>(__ballot(need));
        if (need) words[pos + __popc(m & gt)] = static_cast<uint16_t>(x);
        const uint32_t xr = need ? x >> 16 : x;
        pos += __popc(m);
        const uint32_t xn = rans_next(xr, f, bit ? rcp1 : rcp0, bit ? f0 : 0u);
        x = act ? xn : xr;
      };
      for (uint32_t g = (K - 1) & ~31u;; g -= 32) {    // lane i: the word of step g + i
        const uint32_t w32 = g + lane < K ? bits[g + lane] : 0u;
        if (32 * (g + 32) <= J.nbits) {
#pragma unroll
          for (int i = 31; i >= 0; --i) step(__builtin_amdgcn_readlane(w32, i), true);
        } else {
          for (uint32_t i = K - g; i-- > 0;)
            step(__builtin_amdgcn_readlane(w32, i), 32 * (g + i) + lane < J.nbits);
        }
        if (g == 0) break;
      }
    }
    pos = __builtin_amdgcn_readfirstlane(pos);         // for the lanes that ran no steps
    __builtin_amdgcn_fence(__ATOMIC_ACQ_REL, "agent");
    __builtin_amdgcn_wave_barrier();
    // reverse the pushed words in place: decoder order
    for (uint32_t i = lane; i < pos / 2; i += kWaveE) {
      const uint16_t a = words[i], c = words[pos - 1 - i];
      words[i] = c;
      words[pos - 1 - i] = a;
    }
    if (lane == 0) *reinterpret_cast<uint32_t *>(slot) = pos;
    if (lane < kRansLanes) reinterpret_cast<uint32_t *>(slot)[1 + lane] = x;
    const uint32_t used = kChunkHdr + 2 * pos, size = (used + 3) & ~3u;
    if (lane < size - used) slot[used + lane] = 0;
    if (lane == 0) sizes[j] = size;
    __builtin_amdgcn_wave_barrier();
  }
}

// Byte tANS coding of the chunk jobs (ans_mode 3, Sec. 5.2), a half-wave
// per chunk (persistent over pairs of jobs).  Cursor l of a chunk codes its
// bytes l, l + 32, ... (XOR 0xFF when the marker says complemented) last
// first, from state 2^11: with n = norm(b), the step emits the low nb bits
// of the state, nb the smallest count with (state >> nb) < 2n (11 - k or
// 10 - k for 2^k <= n < 2^(k+1)), and moves to 2^11 + the (state >> nb) -
// n'th state of b.  A first pass finds the cursor's bit count; its stream
// starts after the 128-byte header and the streams of the cursors before it,
// and a second pass writes the bits backwards from the stream's end (the
// decoder reads step 0's bits first).  The table (norm, first, state) sits
// in LDS, reloaded when a half's table changes.
constexpr uint32_t kFseEncNT = 256;
__global__ __launch_bounds__(kFseEncNT) void k_fse_enc(const RansJob *jobs, const Totals *tot,
                                                       const uint32_t *bmp, const uint16_t *enc,
                                                       uint8_t *slots, uint32_t *sizes, uint32_t *err) {
  __shared__ uint16_t tabs[kFseEncNT / kWaveE][2][kFseEncWords];
  const uint32_t lane = __lane_id(), half = lane >> 5, hl = lane & 31;
  const uint32_t wave = threadIdx.x >> 6;
  const uint64_t njobs = tot->chunks;
  const uint64_t nwaves = static_cast<uint64_t>(gridDim.x) * (kFseEncNT / kWaveE);
  uint16_t *E = tabs[wave][half];
  uint32_t loaded = 0;
  for (uint64_t pr = blockIdx.x * (kFseEncNT / kWaveE) + wave; 2 * pr < njobs; pr += nwaves) {
    const uint64_t j = 2 * pr + half;
    const bool has = j < njobs;
    RansJob J{};
    if (has) J = jobs[j];
    const uint32_t t = has ? J.p1q & 0x7F : 0u;
    const uint32_t flip = (J.p1q & 0x80) ? 0xFFu : 0u;
    const uint32_t ta = __builtin_amdgcn_readlane(t, 0), tb = __builtin_amdgcn_readlane(t, 32);
    const uint32_t la = __builtin_amdgcn_readlane(loaded, 0), lb = __builtin_amdgcn_readlane(loaded, 32);
    const bool ra = ta && ta != la, rb = tb && tb != lb;
    if (ra || rb) {
      if (half ? rb : ra) {
        const uint4 *src = reinterpret_cast<const uint4 *>(enc + static_cast<uint64_t>(t - 1) * kFseEncWords);
        uint4 *dst = reinterpret_cast<uint4 *>(E);
        constexpr uint32_t n16 = kFseEncWords * 2 / 16;
        for (uint32_t i = hl; i < n16; i += 32) dst[i] = src[i];
        loaded = t;
      }
      wave_sync();
    }
    const uint16_t *norm = E, *first = E + 256, *state = E + 512;
    const uint8_t *bm = reinterpret_cast<const uint8_t *>(bmp + J.bmp_word);
    const uint32_t cb = (J.nbits + 7) >> 3;
    const uint32_t steps = has && cb > hl ? (cb - hl + 31) >> 5 : 0u;
    // 8 steps from i0 on, last first: their bytes, then the tables' entries of
    // the bytes, are read before the first step, so that the chain of states
    // waits for one table read a step
    auto steps8 = [&](uint32_t i0, uint32_t &x, auto &&emit) {
      uint32_t b[8], n[8], f[8];
#pragma unroll
      for (int e = 0; e < 8; ++e) b[e] = bm[hl + 32 * (i0 + e < steps ? i0 + e : 0u)] ^ flip;
#pragma unroll
      for (int e = 0; e < 8; ++e) {
        n[e] = norm[b[e]];
        f[e] = first[b[e]];
      }
#pragma unroll
      for (int e = 7; e >= 0; --e) {
        const uint32_t k = 31 - __builtin_clz(n[e] | 1u);
        const uint32_t nb = kFseLog - k - (x < (n[e] << (kFseLog - k)) ? 1u : 0u);
        if (i0 + e < steps) {
          emit(x, nb);
          x = kFseSize + state[f[e] + (x >> nb) - n[e]];
        }
      }
    };
    // pass 1: the cursor's bit count and final state
    uint32_t x = kFseSize, tbits = 0;
    for (uint32_t i = (steps + 7) & ~7u; i != 0; i -= 8)
      steps8(i - 8, x, [&](uint32_t, uint32_t nb) { tbits += nb; });
    const uint32_t len = (tbits + 7) >> 3;
    if (len > 0xFFFF) atomicCAS(err, 0u, kErrUnsupported);
    uint32_t incl = wave_incl_scan(len);
    const uint32_t lo = __builtin_amdgcn_readlane(incl, 31), all = __builtin_amdgcn_readlane(incl, 63);
    if (half) incl -= lo;
    const uint32_t total = half ? all - lo : lo;     // stream bytes of this half's chunk
    uint8_t *slot = slots + J.slot;
    uint8_t *sp = slot + kFseChunkHdr + (incl - len);
    // pass 2: the same steps, bits written from the stream's end backwards
    uint32_t acc = 0, accn = 8 * len - tbits, top = len, x2 = kFseSize;
    for (uint32_t i = (steps + 7) & ~7u; i != 0; i -= 8)
      steps8(i - 8, x2, [&](uint32_t xs, uint32_t nb) {
        acc = (acc << nb) | (xs & ((1u << nb) - 1));
        accn += nb;
        while (accn >= 8) {
          --top;
          sp[top] = static_cast<uint8_t>(acc >> (accn - 8));
          accn -= 8;
        }
      });
    if (has) {
      reinterpret_cast<uint16_t *>(slot)[hl] = static_cast<uint16_t>(x - kFseSize);
      reinterpret_cast<uint16_t *>(slot)[kFseLanes + hl] = static_cast<uint16_t>(len);
      const uint32_t used = kFseChunkHdr + total, size = (used + 3) & ~3u;
      if (hl < size - used) slot[used + hl] = 0;
      if (hl == 0) sizes[j] = size;
    }
  }
}

// Size of a block with its entropy-coded nodes (one wave): header, raw
// bodies, then every rANS node at a multiple of 4 bytes with its 8-byte header
// and its chunks, whose sizes are multiples of 4.  The chunks of a block lie in
// node order, so a chunk's place is the sum of the chunks before it and 8
// bytes per node up to its own; it goes to the chunk's job, comp_size to the
// header.
__device__ void block_size(BlockLay &L, RansJob *jobs, const uint32_t *sizes, uint8_t *H) {
  const uint32_t lane = __lane_id(), nch = L.n_chunks;
  uint32_t off = L.hlen + L.raw_bytes;
  if (nch) off = (off + 3) & ~3u;
  for (uint32_t k0 = 0; k0 < nch; k0 += kWaveE) {
    const uint64_t j = L.chunk0 + k0 + lane;
    const bool has = k0 + lane < nch;
    const uint32_t sz = has ? sizes[j] : 0u, inc = wave_incl_scan(sz);
    if (has) jobs[j].dst = off + inc - sz + 8 * (jobs[j].rnode + 1);
    off += __builtin_amdgcn_readlane(inc, 63);
  }
  off += 8 * L.n_rnodes;
  if (lane == 0) {
    L.comp = off;
    *reinterpret_cast<uint32_t *>(H) = off;
  }
}

__global__ __launch_bounds__(256) void k_sizes(BlockLay *lay, RansJob *jobs, const uint32_t *sizes, uint32_t nb,
                                               uint8_t *hdr) {
  const uint32_t b = blockIdx.x * (256 / kWaveE) + __builtin_amdgcn_readfirstlane(threadIdx.x >> 6);
  if (b < nb) block_size(lay[b], jobs, sizes, hdr + static_cast<uint64_t>(b) * kHdrStride);
}

// Stream offsets of the blocks (one workgroup): each block starts at a
// multiple of 4 bytes after the header and the two offset tables.  Up to
// kTailBlocks blocks their sizes are found here too (4 rounds of 16 waves;
// with more blocks the rounds would outlast a launch of k_sizes).  Then the
// call's result.
__global__ __launch_bounds__(kScanNT) void k_scan2(BlockLay *lay, RansJob *jobs, const uint32_t *sizes, uint32_t nb,
                                                   uint8_t *hdr, Totals *tot, uint32_t *err, Result res) {
  __shared__ uint64_t part[kScanNT / kWaveE];
  const uint32_t tid = threadIdx.x;
  if (nb <= kTailBlocks) {
    for (uint32_t b = __builtin_amdgcn_readfirstlane(tid >> 6); b < nb; b += kScanNT / kWaveE)
      block_size(lay[b], jobs, sizes, hdr + static_cast<uint64_t>(b) * kHdrStride);
    __syncthreads();
  }
  uint64_t run = stream_tables(nb);
  for (uint64_t b0 = 0; b0 < nb; b0 += kScanNT) {
    const uint64_t b = b0 + tid;
    uint64_t all;
    const uint64_t x = block_excl_scan(b < nb ? (static_cast<uint64_t>(lay[b].comp) + 3) & ~3ull : 0ull, part, &all);
    if (b < nb) lay[b].out_off = run + x;
    run += all;
  }
  if (tid == 0) {
    tot->out_bytes = run;
    finish(run, err, res);
  }
}

// What the stream's header says.
struct StreamOpts {
  uint64_t n;
  uint32_t bs, max_len, chunk_log2, version;   // version (1 or 2) | flags << 16
};

// Stream header and the two offset tables (block offsets, scratch-word
// offsets), by threads 0 .. nb of a grid.
__device__ void stream_head(uint64_t t, const BlockLay *lay, const Totals *tot, uint32_t nb, const StreamOpts &o,
                            uint8_t *out) {
  uint64_t *boff = reinterpret_cast<uint64_t *>(out + kHeaderBytes);
  uint64_t *aoff = boff + nb + 1;
  if (t <= nb) {
    boff[t] = t < nb ? lay[t].out_off : tot->out_bytes;
    aoff[t] = t < nb ? lay[t].ans0 : tot->ans_words;
  }
  if (t == 0) {
    uint32_t *h = reinterpret_cast<uint32_t *>(out);
    h[0] = kMagic;
    h[1] = o.version;
    h[2] = static_cast<uint32_t>(o.n);
    h[3] = static_cast<uint32_t>(o.n >> 32);
    h[4] = o.bs;
    h[5] = nb;
    h[6] = (o.max_len & 255) | ((o.chunk_log2 & 255) << 8);
    h[7] = 0;
    h[8] = static_cast<uint32_t>(tot->ans_words);
    h[9] = static_cast<uint32_t>(tot->ans_words >> 32);
    h[10] = 0;
    h[11] = 0;
  }
}

// Block header and raw bodies of block b, as aligned 4-byte words (words
// [s kAsmSeg, (s + 1) kAsmSeg) of them): a word inside the raw bodies is a
// byte funnel of two image words, words at the edges are built byte by byte
// (bytes past the raw bodies are zero: the padding before the first rANS body
// or the next block).  Without an image (IMG false) the bodies are zeroed.
template <bool IMG>
__device__ void block_words(uint32_t b, uint32_t s, const BlockLay *lay, const uint8_t *hdr, const uint8_t *imgb,
                            uint8_t *out) {
  const BlockLay &L = lay[b];
  const uint32_t hlen = L.hlen;
  const uint64_t used = static_cast<uint64_t>(hlen) + L.raw_bytes;
  const uint64_t W = (used + 3) / 4;
  const uint64_t w0 = static_cast<uint64_t>(s) * kAsmSeg;
  if (w0 >= W) return;
  const uint64_t w1 = w0 + kAsmSeg < W ? w0 + kAsmSeg : W;
  const uint8_t *H = hdr + static_cast<uint64_t>(b) * kHdrStride;
  const uint8_t *img = imgb + L.img_off;
  const uint32_t *img32 = reinterpret_cast<const uint32_t *>(imgb);
  uint32_t *o32 = reinterpret_cast<uint32_t *>(out + L.out_off);
#pragma unroll 8
  for (uint64_t q = w0 + threadIdx.x; q < w1; q += 256) {
    const uint64_t x0 = 4 * q;
    uint32_t w = 0;
    if (x0 + 4 <= hlen) {
      w = *reinterpret_cast<const uint32_t *>(H + x0);
    } else if (x0 >= hlen && x0 + 4 <= used) {
      if (IMG) {
        const uint64_t so = L.img_off + (x0 - hlen);
        w = __builtin_amdgcn_alignbyte(img32[(so >> 2) + 1], img32[so >> 2], static_cast<uint32_t>(so & 3));
      }
    } else {
      for (uint32_t e = 0; e < 4; ++e) {
        const uint64_t x = x0 + e;
        const uint32_t v = x < hlen ? H[x] : IMG && x < used ? img[x - hlen] : 0u;
        w |= v << (8 * e);
      }
    }
    o32[q] = w;
  }
}

// Streams without entropy-coded nodes: the stream's and the blocks' headers,
// and zeros for the bits that the split kernel writes straight into the
// bodies.  Nothing is written past out_cap.
__global__ __launch_bounds__(256) void k_head(const BlockLay *lay, const Totals *tot, uint32_t nb, uint32_t segs,
                                              StreamOpts o, const uint8_t *hdr, uint8_t *out, uint64_t out_cap) {
  if (tot->out_bytes > out_cap) return;
  stream_head(blockIdx.x * 256ull + threadIdx.x, lay, tot, nb, o, out);
  block_words<false>(blockIdx.x / segs, blockIdx.x % segs, lay, hdr, nullptr, out);
}

// Streams with entropy-coded nodes: the first nb * segs workgroups write the
// headers and the raw bodies from the images; in the others a wave per chunk
// copies its slot into the block, and the first chunk of a node also writes
// the node's 8-byte body header (its bodies end where the next node's header
// or the block does).
__global__ __launch_bounds__(256) void k_assemble(const BlockLay *lay, const Totals *tot, uint32_t nb, uint32_t segs,
                                                  StreamOpts o, const uint8_t *hdr, const uint8_t *imgb,
                                                  const RansNode *rnodes, const RansJob *jobs,
                                                  const uint32_t *sizes, const uint8_t *slots, uint8_t *out,
                                                  uint64_t out_cap) {
  if (tot->out_bytes > out_cap) return;
  stream_head(blockIdx.x * 256ull + threadIdx.x, lay, tot, nb, o, out);
  if (blockIdx.x < nb * segs) {
    block_words<true>(blockIdx.x / segs, blockIdx.x % segs, lay, hdr, imgb, out);
    return;
  }
  const uint32_t lane = __lane_id();
  const uint64_t njobs = tot->chunks;
  const uint64_t nwaves = static_cast<uint64_t>(gridDim.x - nb * segs) * (256 / kWaveE);
  for (uint64_t j = (blockIdx.x - nb * segs) * (256 / kWaveE) + (threadIdx.x >> 6); j < njobs; j += nwaves) {
    const RansJob J = jobs[j];
    const BlockLay &L = lay[J.block];
    uint8_t *dst = out + L.out_off + J.dst;
    if (J.first && lane == 0) {
      const uint32_t end = J.rnode + 1 < L.n_rnodes
                               ? jobs[L.chunk0 + rnodes[255ull * J.block + J.rnode + 1].ch0].dst - 8
                               : L.comp;
      uint32_t *h = reinterpret_cast<uint32_t *>(dst - 8);
      h[0] = J.p1q;                                    // p1q u16, pad u16
      h[1] = end - J.dst;
    }
    const uint32_t *src = reinterpret_cast<const uint32_t *>(slots + J.slot);
    uint32_t *d32 = reinterpret_cast<uint32_t *>(dst);
    const uint32_t nw = sizes[j] / 4;
    for (uint32_t i = lane; i < nw; i += kWaveE) d32[i] = src[i];
  }
}

// The stream of an empty input: header and the two one-entry tables.
struct EmptyStream {
  uint32_t w[16];
};
__global__ void k_empty(EmptyStream h, uint8_t *out, uint64_t out_cap, uint64_t *d_len, int32_t *d_status) {
  const uint32_t t = threadIdx.x;
  const bool fits = out_cap >= sizeof(h.w);
  if (t < 16 && fits) reinterpret_cast<uint32_t *>(out)[t] = h.w[t];
  if (t == 0) {
    *d_len = sizeof(h.w);
    *d_status = fits ? PIVCO_OK : PIVCO_E_CAPACITY;
  }
}

// ---------------------------------------------------------------------------
// host side
// ---------------------------------------------------------------------------
inline uint64_t align_up(uint64_t x, uint64_t a) { return (x + a - 1) / a * a; }

bool opts_ok(const pivco_encode_opts *o) {
  return o && o->block_size >= 1 && o->block_size <= (1u << 30) && o->max_len >= 1 &&
         o->max_len <= kMaxLenGpu && o->ans_mode <= 3 && o->rans_chunk_log2 >= 5 &&
         o->rans_chunk_log2 <= 24 && (o->ans_mode != 3 || o->rans_chunk_log2 >= 8) &&
         o->tree_shape <= 1 && o->reserved == 0;
}

// Large inputs fill the chip with either slice; the larger halves the
// histogram rows and the words that two slices share (256 MiB Zipf: 4 Ki / 8 Ki
// / 16 Ki 2.24 / 2.27 / 2.24 ms a call; 64 MiB very skewed 0.661 / 0.653 /
// 0.667 ms).  Below 8 MiB (1024 large slices, 4 a CU) the smaller one gives
// more workgroups: one 64 KiB block is 16 of them.
// The split's threads (launch_split): up to 256 small slices, one a CU, run
// with 1024 threads, 4 chunks a wave (64 KiB: 18 us, 22 with 256 threads);
// more of them with 256, so that several share a CU.
uint32_t slice_of(uint64_t n, uint32_t block_size) {
  return n >= (8ull << 20) && block_size >= kSliceLarge ? kSliceLarge : kSliceSmall;
}

void launch_split(uint32_t slice, bool flat, uint32_t grid, hipStream_t s, const uint8_t *in, const EncBlock *eb,
                  const BlockLay *lay, uint32_t nb, uint32_t spb, const uint32_t *pre, const uint32_t *hist,
                  uint32_t *img, uint32_t *rbm, const Totals *direct, uint64_t out_cap, const RansNode *rn,
                  uint32_t chunk_log2, RansJob *jobs) {
  auto go = [&](auto kernel, uint32_t nt) {
    hipLaunchKernelGGL(kernel, dim3(grid), dim3(nt), 0, s, in, eb, lay, nb, spb, pre, hist, img, rbm, direct, out_cap,
                       rn, chunk_log2, jobs);
  };
  if (slice == kSliceLarge) {
    if (flat) go(k_split<512, kSliceLarge, true>, 512);
    else go(k_split<512, kSliceLarge, false>, 512);
  } else if (grid > 256) {
    if (flat) go(k_split<256, kSliceSmall, true>, 256);
    else go(k_split<256, kSliceSmall, false>, 256);
  } else {
    if (flat) go(k_split<1024, kSliceSmall, true>, 1024);
    else go(k_split<1024, kSliceSmall, false>, 1024);
  }
}

struct WsLayout {
  uint64_t hist, slh, eb, lay, rnodes, hdr, img, rbm, jobs, sizes, slots, tot, stat, total;
};

// Sizes from n and the options alone (the data is not known yet): every
// area is bounded by the code-length limit and the block count.  A block's tables
// are kept so small that no n and options need more than when the lengths (260
// bytes a block), codes (3520) and, without entropy-coded nodes too, an image lay
// here: a workspace of that size still serves.
WsLayout ws_layout(uint64_t n, const pivco_encode_opts *o) {
  WsLayout L{};
  const uint64_t nb = div_up(n, o->block_size);
  // rows for the small slice also where the large one is taken, so that the
  // workspace of a longer input holds every shorter one
  const uint64_t spb = div_up(std::min<uint64_t>(n, o->block_size), kSliceSmall);
  const uint64_t C = 1ull << o->rans_chunk_log2;
  const uint64_t bits = n * o->max_len;
  const uint64_t chunks = o->ans_mode ? bits / C + nb * 255 + 1 : 0;
  uint64_t x = 0;
  L.hist = x; x = align_up(x + nb * 1024 + 16, 256);
  L.slh = x; x = align_up(x + nb * spb * 1024 + 16, 256);
  L.eb = x; x = align_up(x + nb * sizeof(EncBlock), 256);
  L.lay = x; x = align_up(x + nb * sizeof(BlockLay), 256);
  L.rnodes = x; x = align_up(x + (o->ans_mode ? nb * 255 * sizeof(RansNode) : 0), 256);
  L.hdr = x; x = align_up(x + nb * kHdrStride, 256);
  L.img = x; x = align_up(x + (o->ans_mode ? bits / 8 + nb * (255 + 32) : 0) + 64, 256);
  L.rbm = x; x = align_up(x + (o->ans_mode ? 4 * (bits / 32 + nb * (255 + 4)) : 0) + 64, 256);
  L.jobs = x; x = align_up(x + chunks * sizeof(RansJob), 256);
  L.sizes = x; x = align_up(x + chunks * 4, 256);
  L.slots = x; x = align_up(x + (o->ans_mode ? 2 * bits + chunks * 160 : 0) + 64, 256);
  L.tot = x; x = align_up(x + sizeof(Totals), 256);
  L.stat = x; x = align_up(x + 64, 256);     // error word, then the synchronous call's length and status
  L.total = x;
  return L;
}

#define HIPCHK(x) do { if ((x) != hipSuccess) return PIVCO_E_DEVICE; } while (0)

}  // namespace

uint64_t encode_bound(uint64_t n, const pivco_encode_opts *o) {
  if (!opts_ok(o)) return 0;
  const uint64_t nb = div_up(n, o->block_size);
  const uint64_t C = 1ull << o->rans_chunk_log2;
  const uint64_t bits = n * o->max_len;
  uint64_t b = kHeaderBytes + 16 * (nb + 1) + nb * (12 + 128 + 32 + 4 * 255 + 8);
  if (o->ans_mode == 0) b += bits / 8 + nb * 255;
  else b += 2 * bits + nb * 255 * (12 + 136) + 136 * (bits / C + 1);
  return b;
}

uint64_t encode_workspace(uint64_t n, const pivco_encode_opts *o) {
  if (!opts_ok(o)) return 0;
  return ws_layout(n, o).total;
}

namespace {

// Enqueues a whole encode on s: no host wait.  The stream length and the
// call's status go to d_len and d_status on the device.
pivco_status encode_enqueue(const void *d_in, uint64_t n, void *d_out, uint64_t out_cap, uint64_t *d_len,
                            int32_t *d_status, const pivco_encode_opts *o, void *d_ws, uint64_t ws_bytes,
                            hipStream_t s) {
  if (!opts_ok(o) || (n && !d_in) || !d_out || !d_len || !d_status) return PIVCO_E_ARG;
  if ((reinterpret_cast<uintptr_t>(d_in) & 15) || (reinterpret_cast<uintptr_t>(d_out) & 15))
    return PIVCO_E_ARG;
  if (o->tree && !tree_is_complete(o->tree->code_len, o->max_len)) return PIVCO_E_ARG;
  const uint64_t bs = o->block_size;
  const uint64_t nb64 = div_up(n, bs);
  const uint32_t slice = slice_of(n, o->block_size);
  const uint64_t spb64 = div_up(std::min(n, bs), slice);
  if (nb64 > 0xFFFFFFFFull || nb64 * spb64 > 0x7FFFFFFFull) return PIVCO_E_ARG;
  const uint32_t nb = static_cast<uint32_t>(nb64), spb = static_cast<uint32_t>(spb64);
  const uint32_t flags = o->ans_mode == 3 ? 1u : 0u;
  const uint32_t version = o->tree_shape ? 2u : 1u;
  uint8_t *out = static_cast<uint8_t *>(d_out);
  if (nb == 0) {                         // header and the two one-entry tables
    EmptyStream h{};
    h.w[0] = kMagic;
    h.w[1] = version | (flags << 16);
    h.w[4] = static_cast<uint32_t>(bs);
    h.w[6] = (o->max_len & 255) | ((o->rans_chunk_log2 & 255) << 8);
    h.w[12] = static_cast<uint32_t>(sizeof(h.w));     // block_off[0] = the stream size
    hipLaunchKernelGGL(k_empty, dim3(1), dim3(64), 0, s, h, out, out_cap, d_len, d_status);
    HIPCHK(hipGetLastError());
    return PIVCO_OK;
  }
  const WsLayout L = ws_layout(n, o);
  if (ws_bytes < L.total || !d_ws) return PIVCO_E_CAPACITY;
  const FseTables *ft = nullptr;
  if (o->ans_mode == 3 && !(ft = fse_tables())) return PIVCO_E_DEVICE;   // copied once per device
  uint8_t *ws = static_cast<uint8_t *>(d_ws);
  const uint8_t *in = static_cast<const uint8_t *>(d_in);
  Totals *dtot = reinterpret_cast<Totals *>(ws + L.tot);
  BlockLay *dlay = reinterpret_cast<BlockLay *>(ws + L.lay);
  EncBlock *deb = reinterpret_cast<EncBlock *>(ws + L.eb);
  RansNode *drn = reinterpret_cast<RansNode *>(ws + L.rnodes);
  RansJob *djobs = reinterpret_cast<RansJob *>(ws + L.jobs);
  uint32_t *dsizes = reinterpret_cast<uint32_t *>(ws + L.sizes);
  uint32_t *derr = reinterpret_cast<uint32_t *>(ws + L.stat);

  // 1. histograms of the blocks and of their slices.  The areas that the
  // split kernel ORs into are cleared beside it while their bound is small (a
  // launch costs more than clearing 32 MiB, 7 us, that the data may not need);
  // larger ones to their size, once that is known.
  const bool ans = o->ans_mode != 0;
  const Result res{out_cap, d_len, d_status};
  uint32_t *dh = reinterpret_cast<uint32_t *>(ws + L.hist);
  uint32_t *dslh = reinterpret_cast<uint32_t *>(ws + L.slh);
  uint32_t *dimg = reinterpret_cast<uint32_t *>(ws + L.img);
  uint32_t *drbm = reinterpret_cast<uint32_t *>(ws + L.rbm);
  const uint64_t area = L.jobs - L.img;        // both areas, 256-byte multiples
  const bool early = area <= (32ull << 20);
  hipLaunchKernelGGL(k_hist, dim3(nb * spb), dim3(256), 0, s, in, n, static_cast<uint32_t>(bs), slice, spb, dh, dslh,
                     derr, reinterpret_cast<uint4 *>(dimg), ans && early ? area / 16 : 0ull);
  HIPCHK(hipGetLastError());
  if (spb > kPrefixRows)
    hipLaunchKernelGGL(k_slice_prefix_wide, dim3(16 * nb), dim3(1024), 0, s, dslh, spb, dh);
  else if (spb > 1)
    hipLaunchKernelGGL(k_slice_prefix, dim3(nb), dim3(256), 0, s, dslh, spb, dh);

  // 2. code lengths (package-merge per block, or the supplied tree), layout
  pivco_tree tree{};
  if (o->tree) tree = *o->tree;
  const bool few = nb <= kFewBlocks;
  hipLaunchKernelGGL(few ? k_code<512> : k_code<256>, dim3(nb), dim3(few ? 512 : 256), 0, s, dh, nb, n, static_cast<uint32_t>(bs), o->max_len, tree,
                     o->tree ? 1u : 0u, o->ans_mode, o->rans_chunk_log2, o->tree_shape,
                     ft ? ft->dmax : nullptr, deb, dlay, drn, ws + L.hdr, derr, dtot, res);
  HIPCHK(hipGetLastError());

  // 3. offsets (one block: found by k_code)
  if (nb > 1) hipLaunchKernelGGL(k_scan, dim3(1), dim3(kScanNT), 0, s, dlay, nb, o->ans_mode, dtot, derr, res);
  if (ans && !early) hipLaunchKernelGGL(k_zero_areas, dim3(4096), dim3(256), 0, s, dimg, drbm, dtot);
  HIPCHK(hipGetLastError());

  const StreamOpts so{n, static_cast<uint32_t>(bs), o->max_len, o->rans_chunk_log2, version | (flags << 16)};
  const uint64_t max_words = (kHdrStride + std::min<uint64_t>(n, bs) * o->max_len / 8 + 255 + 4) / 4 + 1;
  const uint32_t segs = static_cast<uint32_t>(div_up(max_words, kAsmSeg));
  if (static_cast<uint64_t>(nb) * segs > 0x7FFFF000ull) return PIVCO_E_UNSUPPORTED;
  if (!ans) {
    // 4. headers, then the bitmaps straight into the stream (nothing is
    // written when it would not fit)
    hipLaunchKernelGGL(k_head, dim3(nb * segs), dim3(256), 0, s, dlay, dtot, nb, segs, so, ws + L.hdr, out, out_cap);
    launch_split(slice, o->tree_shape != 0, nb * spb, s, in, deb, dlay, nb, spb, dslh, dh,
                 reinterpret_cast<uint32_t *>(out), nullptr, dtot, out_cap, drn, o->rans_chunk_log2, nullptr);
    HIPCHK(hipGetLastError());
    return PIVCO_OK;
  }

  // 4. bitmaps, and the entropy-coded chunk jobs
  launch_split(slice, o->tree_shape != 0, nb * spb, s, in, deb, dlay, nb, spb, dslh, dh, dimg, drbm, nullptr, out_cap,
               drn, o->rans_chunk_log2, djobs);
  HIPCHK(hipGetLastError());

  // 5. entropy-coded chunks (at most this many: a grid for them all, or one
  // that strides over the list)
  const uint64_t chunks = n * o->max_len / (1ull << o->rans_chunk_log2) + nb64 * 255 + 1;
  const uint32_t cgrid = static_cast<uint32_t>(std::min<uint64_t>(2048, div_up(chunks, 4)));
  if (ft)
    hipLaunchKernelGGL(k_fse_enc, dim3(cgrid), dim3(kFseEncNT), 0, s, djobs, dtot, drbm, ft->enc,
                       ws + L.slots, dsizes, derr);
  else
    hipLaunchKernelGGL(k_rans_enc, dim3(cgrid), dim3(256), 0, s, djobs, dtot, drbm, ws + L.slots, dsizes);
  HIPCHK(hipGetLastError());

  // 6. sizes and offsets
  if (nb > kTailBlocks)
    hipLaunchKernelGGL(k_sizes, dim3((nb + 3) / 4), dim3(256), 0, s, dlay, djobs, dsizes, nb, ws + L.hdr);
  hipLaunchKernelGGL(k_scan2, dim3(1), dim3(kScanNT), 0, s, dlay, djobs, dsizes, nb, ws + L.hdr, dtot, derr, res);

  // 7. the stream (nothing is written when it would not fit)
  hipLaunchKernelGGL(k_assemble, dim3(nb * segs + cgrid), dim3(256), 0, s, dlay, dtot, nb, segs, so, ws + L.hdr,
                     ws + L.img, drn, djobs, dsizes, ws + L.slots, out, out_cap);
  HIPCHK(hipGetLastError());
  return PIVCO_OK;
}

}  // namespace

pivco_status encode_stream_async(const void *d_in, uint64_t n, void *d_out, uint64_t out_cap,
                                 uint64_t *d_out_len, int32_t *d_status, const pivco_encode_opts *o,
                                 void *d_ws, uint64_t ws_bytes, hipStream_t s) {
  return encode_enqueue(d_in, n, d_out, out_cap, d_out_len, d_status, o, d_ws, ws_bytes, s);
}

pivco_status encode_stream(const void *d_in, uint64_t n, void *d_out, uint64_t out_cap,
                           uint64_t *h_out_len, const pivco_encode_opts *o, void *d_ws,
                           uint64_t ws_bytes, hipStream_t s) {
  if (!opts_ok(o) || !h_out_len || !d_ws) return PIVCO_E_ARG;
  const WsLayout L = ws_layout(n, o);
  if (ws_bytes < L.total) return PIVCO_E_CAPACITY;
  // the result words sit in the workspace's status area
  uint8_t *res = static_cast<uint8_t *>(d_ws) + L.stat + 16;
  uint64_t *d_len = reinterpret_cast<uint64_t *>(res);
  int32_t *d_st = reinterpret_cast<int32_t *>(res + 8);
  const pivco_status st = encode_enqueue(d_in, n, d_out, out_cap, d_len, d_st, o, d_ws, ws_bytes, s);
  if (st) return st;
  struct {
    uint64_t len;
    int32_t status, pad;
  } r{};
  HIPCHK(hipMemcpyAsync(&r, res, 16, hipMemcpyDeviceToHost, s));
  HIPCHK(hipStreamSynchronize(s));
  if (r.status) return static_cast<pivco_status>(r.status);
  *h_out_len = r.len;
  return PIVCO_OK;
}

}  // namespace pivco
