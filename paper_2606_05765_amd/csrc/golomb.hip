// golomb.hip -- PivCo-Golomb (App. G of the paper) on gfx950.
//
// The pivoted layout applied to a unary code: instead of a tree, a list of
// bitmaps, one per code-bit position.  A value v (0..255) is v 0-bits and a
// 1-bit; bitmap k holds, in stream order, the k-th code bit of every value
// >= k, so its 1 bits mark the values equal to k.  Decoding walks the list
// bottom-up, from the last bitmap to the first: at bitmap k a 1 bit gives 0
// and a 0 bit gives 1 + the value the next bitmap holds at that position
// (the appendix's merge_vec_cst_plus1 with constant 0xFF).  Stream format
// "PVG1": a 32-byte header, block offsets, then per block comp_size, n, K
// (bitmaps), the sizes n_1 .. n_{K-1}, and the bitmaps (LSB first).
//
// Encode: k_ghist (per slice, the values >= k) -> k_gprefix (per block, the
// bitmap sizes and places) -> k_gscan (block offsets) -> k_ghead (stream
// header, zeroed blocks) -> k_gsplit (per slice, every value's one 1 bit).
// Nothing is planned on the host; the call waits once, for the length.
// Decode: k_gdecode, one workgroup per block, tiles of 16 values a thread: a
// top-down count gives each bitmap's share of the tile (the 0 bits of one
// bitmap's share are the next one's), then the bottom-up merge: a lane makes
// 16 values from 16 bits, their rank, 4-byte windows of the next bitmap's
// values and one v_perm_b32 per 4 values (selector 0x0C gives the constant
// 0).
#include <hip/hip_runtime.h>

#include <algorithm>
#include <cstring>
#include <vector>

#include "pivco_int.h"

namespace pivco {
namespace {

constexpr uint32_t kGMagic = 0x31475650u;   // "PVG1"
constexpr uint32_t kGHdr = 32;
constexpr int kGW = 64;

// One Golomb job as the decode kernel sees it.
struct GJob {
  const uint8_t *in;
  uint64_t in_len;
  uint8_t *out;
  uint64_t out_cap;
  uint64_t n_total;
  uint32_t n_blocks, block_size;
  uint32_t first;         // its first block among the batch's (jobs in error: none)
  int32_t status;         // its status before any block is decoded
};

// Jobs that travel as arguments of the kernel that stores them: a call of few
// streams copies nothing from the host.
constexpr uint32_t kGArgJobs = 48;
struct GArgs {
  GJob j[kGArgJobs];
};
__global__ void k_ginit(GJob *jobs, uint32_t count, int32_t *status, GArgs a) {
  const uint32_t i = threadIdx.x;
  if (i >= count) return;
  jobs[i] = a.j[i];
  status[i] = a.j[i].status;
}
__global__ void k_gstatus(const GJob *jobs, uint32_t count, int32_t *status) {
  const uint32_t i = blockIdx.x * 256 + threadIdx.x;
  if (i < count) status[i] = jobs[i].status;
}

__device__ __forceinline__ void gset_err(int32_t *status, int32_t e) {
  atomicCAS(reinterpret_cast<int *>(status), 0, e);
}

__device__ __forceinline__ uint32_t g_incl_scan(uint32_t v) {
  v += static_cast<uint32_t>(__builtin_amdgcn_update_dpp(0, static_cast<int>(v), 0x111, 0xf, 0xf, false));
  v += static_cast<uint32_t>(__builtin_amdgcn_update_dpp(0, static_cast<int>(v), 0x112, 0xf, 0xf, false));
  v += static_cast<uint32_t>(__builtin_amdgcn_update_dpp(0, static_cast<int>(v), 0x114, 0xf, 0xf, false));
  v += static_cast<uint32_t>(__builtin_amdgcn_update_dpp(0, static_cast<int>(v), 0x118, 0xf, 0xf, false));
  v += static_cast<uint32_t>(__builtin_amdgcn_update_dpp(0, static_cast<int>(v), 0x142, 0xa, 0xf, false));
  v += static_cast<uint32_t>(__builtin_amdgcn_update_dpp(0, static_cast<int>(v), 0x143, 0xc, 0xf, false));
  return v;
}

__device__ __forceinline__ void g_wave_sync() {
  __builtin_amdgcn_fence(__ATOMIC_RELEASE, "wavefront");
  __builtin_amdgcn_wave_barrier();
  __builtin_amdgcn_fence(__ATOMIC_ACQUIRE, "wavefront");
}

// ---------------------------------------------------------------------------
// encode kernels
// ---------------------------------------------------------------------------
// A value v has one 1 bit, in bitmap v, at the position of the values >= v
// before it; every other bit it adds is 0.  So the encoder never compacts the
// values level by level: it computes that one position per value and sets
// one bit.  The positions come from ranks inside a wave (ballots of v >= k),
// the waves before it in the slice and the slices before it in the block
// (per-slice counts of the values >= k, scanned per block).  Bound by the
// vector instructions of the rank loop, about 25 per level up to the largest
// of a wave's 256 values.  64 Mi values of mean code length 2 in 64 Ki blocks:
// 165 us for the bits and 37 us for the counts, where a workgroup per (block,
// bitmap) passing over the whole block took 3215 us, the counts 138 us and a
// device copy per block header 1440 us; the call 6.1 -> 0.26 ms.
constexpr uint32_t kGES = 8192;             // values per encode slice (one workgroup)
constexpr int kGEN = 256;                   // its threads
constexpr int kGEW = kGEN / kGW;            // its waves
constexpr int kGSteps = kGES / (4 * kGEN);  // steps of 256 values (4 a lane) per wave
constexpr int kGCopies = 16;                // histogram copies: lanes of equal values spread over them
constexpr uint32_t kGStage = 4096;          // staged words: 16 KiB, mean code length up to about 14
constexpr int kGScanNT = 1024;

// One block's size (k_gprefix) and place (k_gscan).
struct GBlk {
  uint64_t comp;          // block bytes
  uint32_t K, pad;        // bitmaps
};

// The 4 consecutive bytes at p + i (no alignment), zero past p + len.
__device__ __forceinline__ uint32_t g_load4(const uint8_t *p, uint32_t i, uint32_t len) {
  uint32_t w = 0;
  if (i + 4 <= len) {
    __builtin_memcpy(&w, p + i, 4);
  } else {
#pragma unroll
    for (uint32_t e = 0; e < 3; ++e)
      if (i + e < len) w |= static_cast<uint32_t>(p[i + e]) << (8 * e);
  }
  return w;
}

// Values present at i (0 to 4) before len.
__device__ __forceinline__ uint32_t g_have(uint32_t i, uint32_t len) {
  return i >= len ? 0u : len - i >= 4 ? 4u : len - i;
}

// Exclusive sum over the workgroup's kGEN threads; *total gets the sum.
template <int NT>
__device__ __forceinline__ uint64_t g_block_scan(uint64_t v, uint64_t *part, uint64_t *total) {
  const uint32_t wave = threadIdx.x >> 6, lane = __lane_id();
  uint64_t x = v;
#pragma unroll
  for (int o = 1; o < kGW; o <<= 1) {
    const uint64_t y = __shfl_up(x, o, kGW);
    if (lane >= static_cast<uint32_t>(o)) x += y;
  }
  if (lane == kGW - 1) part[wave] = x;
  __syncthreads();
  uint64_t before = 0, all = 0;
  for (int w = 0; w < NT / kGW; ++w) {
    const uint64_t p = part[w];
    before += static_cast<uint32_t>(w) < wave ? p : 0u;
    all += p;
  }
  *total = all;
  __syncthreads();
  return before + x - v;
}

// Row blockIdx.x, of `per` slices (see GWs; ONE: of one): entry k = their values
// >= k.
template <bool ONE>
__global__ __launch_bounds__(kGEN) void k_ghist(const uint8_t *in, uint64_t n, uint32_t bs, uint32_t spb,
                                                uint32_t per, uint32_t *rows) {
  __shared__ uint32_t h[kGCopies][257];
  __shared__ uint64_t part[kGEW];
  const uint32_t tid = threadIdx.x;
  for (uint32_t i = tid; i < kGCopies * 257; i += kGEN) (&h[0][0])[i] = 0;
  __syncthreads();
  const uint64_t b = blockIdx.x / spb, sl = blockIdx.x % spb;
  const uint64_t b0 = b * bs, b1 = b0 + bs < n ? b0 + bs : n;
  uint32_t *hc = h[tid % kGCopies];
  for (uint32_t u = 0; u < (ONE ? 1 : per); ++u) {
    const uint64_t s0 = b0 + (ONE ? sl : sl * per + u) * kGES, s1 = s0 + kGES < b1 ? s0 + kGES : b1;
    if (s0 >= s1) break;
    const uint32_t len = static_cast<uint32_t>(s1 - s0);
#pragma unroll
    for (uint32_t t = 0; t < kGES / (4 * kGEN); ++t) {
      const uint32_t i = 4 * (kGEN * t + tid);
      const uint32_t w = g_load4(in + s0, i, len), have = g_have(i, len);
#pragma unroll
      for (uint32_t e = 0; e < 4; ++e)
        if (e < have) atomicAdd(&hc[(w >> (8 * e)) & 255], 1u);
    }
  }
  __syncthreads();
  const uint32_t k = 255 - tid;              // a prefix sum over tid is a suffix sum over k
  uint32_t c = 0;
#pragma unroll
  for (int j = 0; j < kGCopies; ++j) c += h[j][k];
  uint64_t tot;
  const uint64_t ex = g_block_scan<kGEN>(c, part, &tot);
  rows[static_cast<uint64_t>(blockIdx.x) * 256 + k] = static_cast<uint32_t>(ex) + c;
}

// Per block: the slice rows become exclusive prefixes over the slices (16
// rows read before any is rewritten), the totals are the bitmap sizes n_k,
// and a scan of the bitmaps' bytes places them.
__global__ __launch_bounds__(kGEN) void k_gprefix(uint32_t *rows, uint32_t spb, uint32_t *nk, uint64_t *boff,
                                                  GBlk *blk) {
  __shared__ uint64_t part[kGEW];
  const uint64_t b = blockIdx.x;
  const uint32_t k = threadIdx.x;
  uint32_t *row = rows + b * spb * 256 + k;
  uint32_t run = 0, s = 0;
  for (; s + 16 <= spb; s += 16) {
    uint32_t c[16];
#pragma unroll
    for (int j = 0; j < 16; ++j) c[j] = row[256ull * (s + j)];
#pragma unroll
    for (int j = 0; j < 16; ++j) {
      row[256ull * (s + j)] = run;
      run += c[j];
    }
  }
  for (; s < spb; ++s) {
    const uint32_t c = row[256ull * s];
    row[256ull * s] = run;
    run += c;
  }
  const uint32_t K = static_cast<uint32_t>(__syncthreads_count(run != 0));   // n_k never grows with k
  uint64_t body;
  const uint64_t off = g_block_scan<kGEN>((static_cast<uint64_t>(run) + 7) / 8, part, &body);
  const uint64_t hlen = 12 + 4ull * (K ? K - 1 : 0);
  nk[b * 256 + k] = run;
  boff[b * 256 + k] = hlen + off;
  if (k == 0) blk[b] = GBlk{hlen + body, K, 0};
}

// Block offsets in the stream (one workgroup, 1024 blocks at a time).
__global__ __launch_bounds__(kGScanNT) void k_gscan(const GBlk *blk, uint32_t nb, uint64_t *off) {
  __shared__ uint64_t part[kGScanNT / kGW];
  uint64_t run = kGHdr + 8ull * (nb + 1ull);
  for (uint64_t b0 = 0; b0 < nb; b0 += kGScanNT) {
    const uint64_t b = b0 + threadIdx.x;
    const uint64_t c = b < nb ? (blk[b].comp + 3) & ~3ull : 0u;
    uint64_t tot;
    const uint64_t ex = g_block_scan<kGScanNT>(c, part, &tot);
    if (b < nb) off[b] = run + ex;
    run += tot;
  }
  if (threadIdx.x == 0) off[nb] = run;
}

// Stream header and block table; the blocks' words are zeroed (the edges of
// the bitmaps' slices are ORed in).  Nothing is written past out_cap.
__global__ __launch_bounds__(256) void k_ghead(const uint64_t *off, uint32_t nb, uint64_t n, uint32_t bs,
                                               uint32_t *out, uint64_t out_cap) {
  const uint64_t total = off[nb];
  if (total > out_cap) return;
  const uint64_t step = static_cast<uint64_t>(gridDim.x) * blockDim.x;
  const uint64_t t = blockIdx.x * static_cast<uint64_t>(blockDim.x) + threadIdx.x;
  const uint64_t w0 = (kGHdr + 8ull * (nb + 1ull)) / 4;
  if (t == 0) {
    out[0] = kGMagic;
    out[1] = 1;
    out[2] = static_cast<uint32_t>(n);
    out[3] = static_cast<uint32_t>(n >> 32);
    out[4] = bs;
    out[5] = nb;
    out[6] = out[7] = 0;
  }
  for (uint64_t b = t; b <= nb; b += step) reinterpret_cast<uint64_t *>(out + kGHdr / 4)[b] = off[b];
  for (uint64_t w = w0 + t; w < total / 4; w += step) out[w] = 0;
}

struct GEncSmem {
  uint32_t cur[kGEW][256];   // per wave: its values >= k so far; then the staged bit of its first one
  uint64_t gw[256];          // stream word of the slice's first bit in bitmap k
  uint32_t lw[256];          // its staged word
  uint32_t nw[256];          // staged words of bitmap k
  uint64_t part[kGEW];
  uint32_t stage[kGStage];
};

// Bits of one slice.  A wave owns kGSteps * 256 consecutive values, 4 a lane
// per step.  For level k the ballots of v >= k give, by mbcnt, every lane's
// count of values >= k before its own; the values equal to k keep it.  The
// wave's running counts per level sit in LDS.  Then the slice's bitmaps are
// staged in LDS at the alignment of their stream words, one atomicOr per
// value, and go out as words: the first and last word of a bitmap's share
// may belong to a neighbour too and are ORed, the others are stored.  A slice
// of long codes that does not fit the stage sets its bits in the stream.  A
// workgroup with several slices (ONE false) takes them in turn; the loop in every
// workgroup took 172 us for 162.
template <bool ONE>
__global__ __launch_bounds__(kGEN, 5) void k_gsplit(const uint8_t *in, uint64_t n, uint32_t bs, uint32_t spb,
                                                 uint32_t per, const uint32_t *rows, const uint32_t *nk,
                                                 const uint64_t *boff, const GBlk *blk, const uint64_t *off,
                                                 uint32_t nb, uint32_t *out, uint64_t out_cap) {
  __shared__ GEncSmem sm;
  if (off[nb] > out_cap) return;
  const uint32_t tid = threadIdx.x, wave = tid >> 6, lane = __lane_id();
  const uint64_t b = blockIdx.x / spb, sl = blockIdx.x % spb;
  const uint64_t b0 = b * bs, b1 = b0 + bs < n ? b0 + bs : n;
  if (sl == 0) {                              // block header: whole words
    uint32_t *h = out + off[b] / 4;
    const uint32_t K = blk[b].K;
    if (tid == 0) {
      h[0] = static_cast<uint32_t>(blk[b].comp);
      h[1] = static_cast<uint32_t>(b1 - b0);
      h[2] = K;
    } else if (tid < K) {
      h[2 + tid] = nk[b * 256 + tid];
    }
  }
  uint32_t *cur = sm.cur[wave];
  uint32_t done = 0;                          // thread k: bits of level k in this workgroup's earlier slices
  for (uint32_t u = 0; u < (ONE ? 1 : per); ++u) {
    const uint64_t s0 = b0 + (ONE ? sl : sl * per + u) * kGES, s1 = s0 + kGES < b1 ? s0 + kGES : b1;
    if (s0 >= s1) return;
#pragma unroll
    for (int e = 0; e < 4; ++e) cur[kGW * e + lane] = 0;
    g_wave_sync();
    uint32_t vw[kGSteps];                       // 4 values a word
    uint32_t pos[kGSteps][2];                   // two 16-bit positions a word
    const uint32_t len = static_cast<uint32_t>(s1 - s0), i0 = wave * (256 * kGSteps) + 4 * lane;
#pragma unroll
    for (int t = 0; t < kGSteps; ++t) vw[t] = g_load4(in + s0, i0 + 256 * t, len);
#pragma unroll
    for (int t = 0; t < kGSteps; ++t) {
      const uint32_t have = g_have(i0 + 256 * t, len);
      int v[4];
      uint32_t at[4], r[4] = {0, 0, 0, 0};
#pragma unroll
      for (uint32_t e = 0; e < 4; ++e) {
        const uint32_t x = (vw[t] >> (8 * e)) & 255;
        at[e] = cur[x];
        v[e] = e < have ? static_cast<int>(x) : -1;
      }
      g_wave_sync();
      for (int k = 0; k < 256; ++k) {
        uint64_t S[4];
#pragma unroll
        for (int e = 0; e < 4; ++e) S[e] = __ballot(v[e] >= k);
        const uint32_t all = static_cast<uint32_t>(__popcll(S[0]) + __popcll(S[1]) + __popcll(S[2]) + __popcll(S[3]));
        if (all == 0) break;
        uint32_t c = 0;
#pragma unroll
        for (int e = 0; e < 4; ++e)
          c = __builtin_amdgcn_mbcnt_hi(static_cast<uint32_t>(S[e] >> 32),
                                        __builtin_amdgcn_mbcnt_lo(static_cast<uint32_t>(S[e]), c));
#pragma unroll
        for (int e = 0; e < 4; ++e) {
          r[e] = v[e] == k ? c : r[e];
          c += v[e] >= k ? 1u : 0u;
        }
        if (lane == 0) atomicAdd(&cur[k], all);   // no value back: the loop does not wait for it
      }
      g_wave_sync();
      pos[t][0] = (at[0] + r[0]) | (at[1] + r[1]) << 16;
      pos[t][1] = (at[2] + r[2]) | (at[3] + r[3]) << 16;
      // the words as they are, opaque: otherwise the unpacked values and
      // positions of all steps are kept for the placing below, and spilled
      asm volatile("" : "+v"(vw[t]), "+v"(pos[t][0]), "+v"(pos[t][1]));
    }
    __syncthreads();
    uint32_t words = 0, sh = 0, cw[kGEW], cnt = 0;
    uint64_t gb = 0;
    {
      const uint32_t k = tid;
#pragma unroll
      for (int w = 0; w < kGEW; ++w) { cw[w] = sm.cur[w][k]; cnt += cw[w]; }
      if (cnt) {
        gb = 8 * (off[b] + boff[b * 256 + k]) + rows[static_cast<uint64_t>(blockIdx.x) * 256 + k] + (ONE ? 0u : done);
        sh = static_cast<uint32_t>(gb & 31);
        words = (sh + cnt + 31) / 32;
      }
    }
    done += cnt;
    const uint32_t Ks = static_cast<uint32_t>(__syncthreads_count(cnt != 0));
    uint64_t tot;
    const uint32_t lw = static_cast<uint32_t>(g_block_scan<kGEN>(words, sm.part, &tot));
    {
      uint32_t x = 32 * lw + sh;                // below 2^23: at most 8192 * 256 staged bits and the edges
#pragma unroll
      for (int w = 0; w < kGEW; ++w) { sm.cur[w][tid] = x; x += cw[w]; }
      sm.gw[tid] = gb >> 5;
      sm.lw[tid] = lw;
      sm.nw[tid] = words;
    }
    const bool staged = tot <= kGStage;
    if (staged)
      for (uint32_t i = tid; i < tot; i += kGEN) sm.stage[i] = 0;
    __syncthreads();
#pragma unroll
    for (int t = 0; t < kGSteps; ++t) {
      const uint32_t have = g_have(i0 + 256 * t, len);
#pragma unroll
      for (uint32_t e = 0; e < 4; ++e) {
        if (e >= have) continue;
        const uint32_t k = (vw[t] >> (8 * e)) & 255;
        const uint32_t x = cur[k] + ((pos[t][e >> 1] >> (16 * (e & 1))) & 0xFFFF);
        if (staged) atomicOr(&sm.stage[x >> 5], 1u << (x & 31));
        else atomicOr(&out[sm.gw[k] + ((x >> 5) - sm.lw[k])], 1u << (x & 31));
      }
    }
    if (!staged) continue;
    __syncthreads();
    for (uint32_t k = wave; k < Ks; k += kGEW) {
      const uint32_t nw = sm.nw[k], l0 = sm.lw[k];
      uint32_t *dst = out + sm.gw[k];
      for (uint32_t j = lane; j < nw; j += kGW) {
        const uint32_t w = sm.stage[l0 + j];
        if (j == 0 || j == nw - 1) {
          if (w) atomicOr(&dst[j], w);
        } else {
          dst[j] = w;
        }
      }
    }
  }
}

// ---------------------------------------------------------------------------
// decode kernel
// ---------------------------------------------------------------------------
// Workgroups of 1024 threads, tiles of 16384 values, where two a CU hold all
// blocks and some block is longer than a tile of 512 threads: a tile's time is
// its levels' latency, and few blocks leave nothing to hide it behind.  Mean code
// length 2, 512 and 1024 threads: one block of 1 Mi values 1146 and 735 us a call,
// 512 blocks of 64 Ki 152 and 126; 1024 blocks, which 512 threads still hold at
// once, 167 and 186.  Uniform values (mean 128): 512 blocks of 64 Ki 3.47 and 2.44
// ms, 768 3.84 and 4.00.
constexpr uint32_t kGFew = 512, kGNarrow = 16 * 512;
constexpr uint32_t kGWave = 16 * kGW;       // values one wave merges at once

template <int NT>
struct GSmem {
  uint32_t nk[257];          // values reaching bitmap k (n_0 = n, n_K = 0)
  uint32_t cur[257];         // of which decoded by earlier tiles
  uint32_t tv[257];          // of which in this tile
  uint64_t boff[256];        // bitmap k's first byte in the stream
  uint64_t part[NT / kGW];
  uint32_t wsum[2][NT / kGW];
  uint32_t sel[16];
  uint32_t err, depth;
  uint32_t lvl[2][4 * NT + 32] __attribute__((aligned(16)));
};

// Sum over the workgroup of a wave's inclusive scan `inc` (its last lane's),
// and of the waves before this one; one barrier, two slots used in turn.
template <int NT>
__device__ __forceinline__ uint32_t g_waves(GSmem<NT> &sm, uint32_t slot, uint32_t inc, uint32_t *before) {
  const uint32_t wave = threadIdx.x >> 6;
  if (__lane_id() == kGW - 1) sm.wsum[slot][wave] = inc;
  __syncthreads();
  uint32_t b = 0, t = 0;
#pragma unroll
  for (uint32_t w = 0; w < NT / kGW; ++w) {
    const uint32_t x = sm.wsum[slot][w];
    b += w < wave ? x : 0u;
    t += x;
  }
  *before = b;
  return t;
}

// The first n (0 to 16) of 16 bits.
__device__ __forceinline__ uint32_t g_first(uint32_t bits, uint32_t x, uint32_t n) {
  return x >= n ? 0u : n - x >= 16 ? bits : bits & ((1u << (n - x)) - 1);
}

// 16 outputs of a level from 16 bits and the 1 bits before them: 4-byte
// windows of the next level's values at cb + rank, one v_perm_b32 per 4.
template <int NT>
__device__ __forceinline__ void g_merge16(const GSmem<NT> &sm, uint32_t parity, uint32_t x, uint32_t bits, uint32_t r1,
                                          uint32_t o[4]) {
  const uint8_t *lds = reinterpret_cast<const uint8_t *>(&sm);
  uint32_t a[4], s[4], w0[4], w1[4];
  a[0] = static_cast<uint32_t>(reinterpret_cast<const uint8_t *>(sm.lvl[parity]) - lds) + x - r1;
#pragma unroll
  for (int g = 0; g < 4; ++g) {
    const uint32_t m = (bits >> (4 * g)) & 15;
    if (g < 3) a[g + 1] = a[g] + 4 - __popc(m);
    s[g] = sm.sel[m];
  }
#pragma unroll
  for (int g = 0; g < 4; ++g) {
    const uint32_t *q = reinterpret_cast<const uint32_t *>(lds + (a[g] & ~3u));
    w0[g] = q[0];
    w1[g] = q[1];
  }
#pragma unroll
  for (int g = 0; g < 4; ++g) o[g] = __builtin_amdgcn_perm(0u, __builtin_amdgcn_alignbyte(w1[g], w0[g], a[g]), s[g]);
}

// Values of a level to its buffer, plus one (the level above reads them as
// "1 + value"); the root's to the output.
template <int NT>
__device__ __forceinline__ void g_put(GSmem<NT> &sm, int k, uint32_t x, uint32_t n, const uint32_t o[4], uint8_t *out) {
  if (x >= n) return;
  if (k > 0) {
    *reinterpret_cast<uint4 *>(reinterpret_cast<uint8_t *>(sm.lvl[k & 1]) + x) =
        make_uint4(o[0] + 0x01010101u, o[1] + 0x01010101u, o[2] + 0x01010101u, o[3] + 0x01010101u);
  } else if (n - x >= 16) {
    const uint4 v = make_uint4(o[0], o[1], o[2], o[3]);
    __builtin_memcpy(out + x, &v, 16);       // blocks start at any byte
  } else {
    for (uint32_t e = 0; e < n - x; ++e) out[x + e] = static_cast<uint8_t>(o[e >> 2] >> (8 * (e & 3)));
  }
}

// One workgroup per block, tiles of 16 values a thread.  Top-down, the 0 bits of
// a level's share are the next level's share; bottom-up, the merge.  The root's
// bits stay in a register for both directions, wave 0 takes every level of at
// most kGWave values without a barrier.  A level of at most 64 values and all
// below it need no way up: a lane per value follows it down, its place among
// the values still alive a mbcnt of their ballot, each level's bits a 64-bit
// scalar, loaded at the tile's start.  The other levels load their bits in each
// direction.  (Ten levels' bits loaded up front and held in registers spilled 50
// registers past the 64 that 8 waves a SIMD leave: 1024 blocks of 64 Ki values of mean code length
// 2 took 143 us, 104 without; the call 203 and 165, of 16384 blocks of 4 Ki 363 and 259.)
// Bound by the vector instructions of the levels (about 60 per 1024 values)
// and the chain of the deep ones.
template <int NT>
__global__ __launch_bounds__(NT, 8) void k_gdecode(const GJob *jobs, uint32_t njobs, uint32_t nblocks,
                                                   int32_t *status) {
  constexpr uint32_t kGT = 16 * NT;          // values per tile
  __shared__ GSmem<NT> sm;
  const uint32_t tid = threadIdx.x, lane = __lane_id();
  const uint32_t wave = __builtin_amdgcn_readfirstlane(tid >> 6);
  if (blockIdx.x >= nblocks) return;
  uint32_t job = 0;          // the last job whose blocks start at or before this one
  for (uint32_t n = njobs; n > 1;) {
    const uint32_t half = n / 2;
    if (jobs[job + half].first <= blockIdx.x) { job += half; n -= half; }
    else n = half;
  }
  const GJob &J = jobs[job];
  const uint32_t b = blockIdx.x - J.first;
  status += job;
  if (tid < 16) {            // v_perm selectors: byte e takes the next value of
    uint32_t s = 0, z = 0;   // the next bitmap (0 bit) or the constant 0 (1 bit)
    for (int e = 0; e < 4; ++e) {
      const uint32_t bit = (tid >> e) & 1;
      s |= (bit ? 0x0Cu : z) << (8 * e);
      z += 1 - bit;
    }
    sm.sel[tid] = s;
  }
  // the block's header, checked by every thread, and bitmap tid's size and place
  const uint8_t *const in = J.in;
  const uint64_t *tab = reinterpret_cast<const uint64_t *>(in + kGHdr);
  const uint64_t off = tab[b], end = tab[b + 1];
  const uint64_t want = J.n_total - static_cast<uint64_t>(b) * J.block_size < J.block_size
                            ? J.n_total - static_cast<uint64_t>(b) * J.block_size : J.block_size;
  bool bad = off < kGHdr + 8ull * (J.n_blocks + 1ull) || end < off || end > J.in_len || (off & 3) || end - off < 12;
  uint32_t K = 0, n = 0, nk = 0;
  uint64_t hlen = 12;
  const uint8_t *p = in + off;
  uint32_t comp = 0;
  if (!bad) {
    const uint32_t *p32 = reinterpret_cast<const uint32_t *>(p);
    comp = p32[0];
    n = p32[1];
    const uint32_t kw = p32[2];
    K = kw & 0xFFFF;
    hlen = 12 + 4ull * (K ? K - 1 : 0);
    bad = n != want || (kw >> 16) || K > 256 || (n == 0) != (K == 0) || comp < hlen || comp > end - off ||
          ((comp + 3ull) & ~3ull) != end - off;
    if (!bad && tid < K) nk = tid ? p32[2 + tid] : n;
  }
  if (tid < 256) sm.nk[tid] = nk;
  if (tid == 0) { sm.nk[256] = 0; sm.err = 0; }
  uint64_t body;
  const uint64_t bo = g_block_scan<NT>((static_cast<uint64_t>(nk) + 7) / 8, sm.part, &body);
  if (tid < 256) {
    sm.boff[tid] = off + hlen + bo;
    sm.cur[tid] = 0;
    if (!bad && tid && tid < K && nk > sm.nk[tid - 1]) bad = true;
  }
  if (tid == 0) sm.cur[256] = 0;
  if (!bad && hlen + body != comp) bad = true;
  if (__syncthreads_or(bad)) {
    if (tid == 0) gset_err(status, PIVCO_E_CORRUPT);
    return;
  }
  uint8_t *out = J.out + static_cast<uint64_t>(b) * J.block_size;
  // 16 bits of bitmap k, x values after its cursor (zeros where it holds no
  // more); the block ends at a multiple of 4 bytes, so whole words of it are read
  const uint32_t *in32 = reinterpret_cast<const uint32_t *>(in);
  const uint64_t wend = end >> 2;
  auto fetch = [&](uint32_t k, uint32_t x) -> uint32_t {
    const uint32_t c = sm.cur[k];
    if (k >= K || x >= sm.nk[k] - c) return 0u;
    const uint64_t bit = 8 * sm.boff[k] + c + x, q = bit >> 5;
    const uint32_t w0 = in32[q], w1 = q + 1 < wend ? in32[q + 1] : 0u;
    return __builtin_amdgcn_alignbit(w1, w0, static_cast<uint32_t>(bit & 31)) & 0xFFFF;
  };
  const uint32_t x = 16 * tid, xl = 16 * lane;
  for (uint32_t t0 = 0; t0 < n; t0 += kGT) {
    const uint32_t S = n - t0 < kGT ? n - t0 : kGT;
    uint32_t root = fetch(0, x);
    uint32_t w_lo = 0, w_hi = 0, rem = 0;    // level lane: its first 64 bits, values left of it
    auto words64 = [&](uint32_t k) {
      w_lo = w_hi = rem = 0;
      if (k >= K) return;
      const uint32_t c = sm.cur[k];
      rem = sm.nk[k] - c;
      if (rem == 0) return;
      const uint64_t bit = 8 * sm.boff[k] + c, q = bit >> 5;
      const uint32_t a0 = in32[q], a1 = q + 1 < wend ? in32[q + 1] : 0u, a2 = q + 2 < wend ? in32[q + 2] : 0u;
      w_lo = __builtin_amdgcn_alignbit(a1, a0, static_cast<uint32_t>(bit & 31));
      w_hi = __builtin_amdgcn_alignbit(a2, a1, static_cast<uint32_t>(bit & 31));
    };
    if (wave == 0) words64(lane);
    // count
    uint32_t tv = S, kmax = 0;               // kmax: levels with a share in this tile
    bool over = false;
    auto next = [&](uint32_t k, uint32_t ones) {   // level k's share tv is counted
      if (tid == 0) sm.tv[k] = tv;
      kmax = k + 1;
      const uint32_t zeros = tv - ones;
      over |= sm.cur[k + 1] + zeros > sm.nk[k + 1];
      tv = over ? 0u : zeros;
    };
    const uint32_t wave0 = kGWave * wave;    // the wave's first value
    {
      uint32_t bits = 0, pc = 0, inc = 0, before;
      if (wave0 < S) {
        bits = g_first(root, x, S);
        pc = __popc(bits);
        inc = g_incl_scan(pc);
      }
      const uint32_t ones = g_waves(sm, 0, inc, &before);
      root = bits | ((before + inc - pc) << 16);   // with the 1 bits before them
      next(0, ones);
    }
    // the levels wider than a wave
    uint32_t kw = kmax;
    while (tv > kGWave) {
      const uint32_t k = kmax;
      uint32_t inc = 0, before;
      if (wave0 < tv) inc = g_incl_scan(__popc(g_first(fetch(k, x), x, tv)));
      next(k, g_waves(sm, k & 1, inc, &before));
      kw = kmax;
    }
    // one wave takes the rest, down and up again
    if (wave == 0 && tv) {
      const int k0 = static_cast<int>(kmax);
      auto total = [](uint32_t inc) { return static_cast<uint32_t>(__builtin_amdgcn_readlane(static_cast<int>(inc), kGW - 1)); };
      while (tv > kGW) {
        const uint32_t bits = g_first(fetch(kmax, xl), xl, tv);
        next(kmax, total(g_incl_scan(__popc(bits))));
      }
      const int kd = static_cast<int>(kmax);
      if (tv) {                              // at most 64 values: a lane each, straight down
        bool alive = lane < tv;
        uint32_t val = 0, tvs = 0;
        uint32_t k = static_cast<uint32_t>(kd), base = 0;
        while (tv) {
          if (k - base >= kGW) {             // the next 64 levels (the first are loaded)
            if (base + lane >= static_cast<uint32_t>(kd) && base + lane < k) sm.tv[base + lane] = tvs;
            base = k & ~(kGW - 1u);
            words64(base + lane);
          }
          const uint32_t l = k - base;
          if (tv > static_cast<uint32_t>(__builtin_amdgcn_readlane(static_cast<int>(rem), l))) { over = true; break; }
          const uint32_t lo = __builtin_amdgcn_readlane(static_cast<int>(w_lo), l);
          const uint32_t hi = __builtin_amdgcn_readlane(static_cast<int>(w_hi), l);
          const uint64_t am = __ballot(alive);
          const uint32_t idx = __builtin_amdgcn_mbcnt_hi(static_cast<uint32_t>(am >> 32),
                                                         __builtin_amdgcn_mbcnt_lo(static_cast<uint32_t>(am), 0u));
          if (lane == l) tvs = tv;
          const bool one = alive && (((idx & 32 ? hi : lo) >> (idx & 31)) & 1);
          if (one) val = k - static_cast<uint32_t>(kd);
          alive = alive && !one;
          tv = static_cast<uint32_t>(__popcll(__ballot(alive)));
          ++k;
        }
        kmax = k;
        if (base + lane >= static_cast<uint32_t>(kd) && base + lane < k) sm.tv[base + lane] = tvs;
        reinterpret_cast<uint8_t *>(sm.lvl[kd & 1])[lane] = static_cast<uint8_t>(val + 1);
      }
      g_wave_sync();
      for (int k = kd - 1; k >= k0; --k) {
        const uint32_t m = sm.tv[k], bits = g_first(fetch(k, xl), xl, m), pc = __popc(bits);
        uint32_t o[4];
        g_merge16(sm, (k + 1) & 1, xl, bits, g_incl_scan(pc) - pc, o);
        g_put(sm, k, xl, m, o, out + t0);
        g_wave_sync();
      }
      if (lane == 0) {
        sm.depth = kmax;
        if (over) sm.err = static_cast<uint32_t>(PIVCO_E_CORRUPT);
      }
    } else if (tv == 0 && tid == 0) {
      sm.depth = kmax;
      if (over) sm.err = static_cast<uint32_t>(PIVCO_E_CORRUPT);
    }
    __syncthreads();
    kmax = sm.depth;
    if (sm.err) break;
    for (int k = static_cast<int>(kw) - 1; k >= 1; --k) {
      const uint32_t m = sm.tv[k];
      uint32_t bits = 0, pc = 0, inc = 0, before;
      if (wave0 < m) {
        bits = g_first(fetch(k, x), x, m);
        pc = __popc(bits);
        inc = g_incl_scan(pc);
      }
      g_waves(sm, k & 1, inc, &before);
      if (wave0 < m) {
        uint32_t o[4];
        g_merge16(sm, (k + 1) & 1, x, bits, before + inc - pc, o);
        g_put(sm, k, x, m, o, out + t0);
      }
      __syncthreads();
    }
    if (wave0 < S) {
      uint32_t o[4];
      g_merge16(sm, 1, x, root & 0xFFFF, root >> 16, o);
      g_put(sm, 0, x, S, o, out + t0);
    }
    for (uint32_t k = tid; k < kmax; k += NT) sm.cur[k] += sm.tv[k];
    __syncthreads();
  }
  // the whole block consumed every bitmap, and the last one had no 0 bit
  if (!sm.err)
    for (uint32_t k = tid; k < K; k += NT)
      if (sm.cur[k] != sm.nk[k]) atomicCAS(&sm.err, 0u, static_cast<uint32_t>(PIVCO_E_CORRUPT));
  __syncthreads();
  if (tid == 0 && sm.err) gset_err(status, static_cast<int32_t>(sm.err));
}

inline uint64_t galign(uint64_t x, uint64_t a) { return (x + a - 1) / a * a; }

// Encode workspace: rows of `per` slices each, then per block the bitmap sizes,
// their places, the block's size and its offset.
struct GWs {
  uint64_t rows, nk, boff, blk, off, total;
  uint32_t per, spb;      // slices a row, rows per block
};
GWs gws_layout(uint64_t n, uint32_t bs, uint32_t per) {
  GWs L{};
  const uint64_t nb = div_up(n, bs);
  L.per = per;
  L.spb = static_cast<uint32_t>(div_up(std::min<uint64_t>(n, bs), static_cast<uint64_t>(per) * kGES));
  uint64_t x = 0;
  L.rows = x; x = galign(x + nb * L.spb * 1024, 256);
  L.nk = x; x = galign(x + nb * 1024, 256);
  L.boff = x; x = galign(x + nb * 2048, 256);
  L.blk = x; x = galign(x + nb * sizeof(GBlk), 256);
  L.off = x; x = galign(x + 8 * (nb + 1), 256);
  L.total = x;
  return L;
}

// Bytes that have always been enough for an encode: the room of a list of the
// block's bitmaps (24 bytes each, at most 256) and of its header beside its
// counts.  A row per slice takes more than that for blocks past 24 Ki values, so
// an encode with less room than pivco_golomb_encode_workspace asks for takes rows
// of more slices.
uint64_t gws_enough(uint64_t n, uint32_t bs) {
  const uint64_t nb = div_up(n, bs);
  return galign(nb * 1024 + 16, 256) + galign(nb * 256 * 24, 256) +
         galign(kGHdr + 8 * (nb + 1) + nb * (12 + 4 * 255) + 64, 256);
}

// Workgroups of kGEN threads that one launch may have: fewer than 2^32 threads.
constexpr uint64_t kGMaxGrid = ((1ull << 32) - 1) / kGEN;

}  // namespace
}  // namespace pivco

using namespace pivco;

extern "C" {

uint64_t pivco_golomb_encode_bound(uint64_t n, uint32_t block_size) {
  if (block_size == 0) return 0;
  const uint64_t nb = div_up(n, block_size);
  return kGHdr + 8 * (nb + 1) + nb * (12 + 4 * 255 + 256 + 4) + 32 * n;
}

uint64_t pivco_golomb_encode_workspace(uint64_t n, uint32_t block_size) {
  if (block_size == 0) return 0;
  return gws_layout(n, block_size, 1).total;
}

pivco_status pivco_golomb_encode(const void *d_in, uint64_t n, uint32_t block_size, void *d_out,
                                 uint64_t out_cap, uint64_t *h_out_len, void *d_ws, uint64_t ws_bytes,
                                 hipStream_t s) {
  if (!h_out_len || block_size == 0 || (n && !d_in) || !d_out || (reinterpret_cast<uintptr_t>(d_out) & 15))
    return PIVCO_E_ARG;
  const uint64_t nb64 = div_up(n, block_size);
  if (nb64 > 0xFFFFFFFFull) return PIVCO_E_ARG;
  GWs L = gws_layout(n, block_size, 1);
  if (!d_ws || ws_bytes < std::min(L.total, gws_enough(n, block_size))) return PIVCO_E_CAPACITY;
  while (L.spb > 1 && (L.total > ws_bytes || nb64 * L.spb > kGMaxGrid)) L = gws_layout(n, block_size, 2 * L.per);
  if (nb64 * L.spb > 0x7FFFFFFFull) return PIVCO_E_ARG;
  if (nb64 > kGMaxGrid) return PIVCO_E_DEVICE;       // no launch has a workgroup for every block
  const uint32_t nb = static_cast<uint32_t>(nb64), spb = L.spb, per = L.per;
  const uint8_t *in = static_cast<const uint8_t *>(d_in);
  uint8_t *ws = static_cast<uint8_t *>(d_ws);
  uint32_t *rows = reinterpret_cast<uint32_t *>(ws + L.rows), *nk = reinterpret_cast<uint32_t *>(ws + L.nk);
  uint64_t *boff = reinterpret_cast<uint64_t *>(ws + L.boff), *off = reinterpret_cast<uint64_t *>(ws + L.off);
  GBlk *blk = reinterpret_cast<GBlk *>(ws + L.blk);
  uint32_t *out = static_cast<uint32_t *>(d_out);
  if (nb) {
    hipLaunchKernelGGL(per == 1 ? k_ghist<true> : k_ghist<false>, dim3(nb * spb), dim3(kGEN), 0, s, in, n, block_size,
                       spb, per, rows);
    hipLaunchKernelGGL(k_gprefix, dim3(nb), dim3(kGEN), 0, s, rows, spb, nk, boff, blk);
    if (hipGetLastError() != hipSuccess) return PIVCO_E_DEVICE;   // the rest reads what these write
  }
  hipLaunchKernelGGL(k_gscan, dim3(1), dim3(kGScanNT), 0, s, blk, nb, off);
  // the stream is at most the bound: 8 words a thread when it is that large
  const uint64_t most = pivco_golomb_encode_bound(n, block_size) / 4;
  hipLaunchKernelGGL(k_ghead, dim3(static_cast<uint32_t>(std::min<uint64_t>(2048, div_up(most, 2048)))),
                     dim3(256), 0, s, off, nb, n, block_size, out, out_cap);
  if (nb)
    hipLaunchKernelGGL(per == 1 ? k_gsplit<true> : k_gsplit<false>, dim3(nb * spb), dim3(kGEN), 0, s, in, n,
                       block_size, spb, per, rows, nk, boff, blk, off, nb, out, out_cap);
  if (hipGetLastError() != hipSuccess) return PIVCO_E_DEVICE;
  uint64_t total = 0;
  if (hipMemcpyAsync(&total, off + nb, 8, hipMemcpyDeviceToHost, s) != hipSuccess ||
      hipStreamSynchronize(s) != hipSuccess)
    return PIVCO_E_DEVICE;
  if (total > out_cap) return PIVCO_E_CAPACITY;
  *h_out_len = total;
  return PIVCO_OK;
}

uint64_t pivco_golomb_decode_workspace(const pivco_job *h_jobs, uint32_t count, hipStream_t s) {
  if (count && !h_jobs) return 0;
  uint64_t nb = 0;
  for (uint32_t j = 0; j < count; ++j) {
    uint8_t h[kGHdr];
    if (h_jobs[j].in_len < kGHdr || !h_jobs[j].d_in) continue;
    if (hipMemcpy(h, h_jobs[j].d_in, kGHdr, hipMemcpyDeviceToHost) != hipSuccess) return 0;
    uint32_t m = 0, b = 0;
    std::memcpy(&m, h, 4);
    std::memcpy(&b, h + 20, 4);
    if (m == kGMagic) nb += b;
  }
  (void)s;
  return galign(count * sizeof(GJob) + 16, 256) + galign(8 * nb + 16, 256);
}

pivco_status pivco_golomb_decode(const pivco_job *h_jobs, uint32_t count, int32_t *d_status, void *d_ws,
                                 uint64_t ws_bytes, hipStream_t s) {
  if (count && (!h_jobs || !d_status || !d_ws)) return PIVCO_E_ARG;
  std::vector<GJob> jobs(count);
  uint64_t blocks = 0, longest = 0;
  for (uint32_t j = 0; j < count; ++j) {
    const pivco_job &jb = h_jobs[j];
    GJob &g = jobs[j];
    std::memset(&g, 0, sizeof(g));
    g.in = static_cast<const uint8_t *>(jb.d_in);
    g.in_len = jb.in_len;
    g.out = static_cast<uint8_t *>(jb.d_out);
    g.out_cap = jb.out_cap;
    g.first = static_cast<uint32_t>(blocks);
    if (jb.in_len && (!jb.d_in || (reinterpret_cast<uintptr_t>(jb.d_in) & 15))) return PIVCO_E_ARG;
    uint8_t h[kGHdr] = {0};
    if (jb.in_len < kGHdr || hipMemcpy(h, jb.d_in, kGHdr, hipMemcpyDeviceToHost) != hipSuccess) {
      g.status = PIVCO_E_CORRUPT;
      continue;
    }
    uint32_t m = 0, bs = 0, nb = 0;
    uint64_t n = 0;
    std::memcpy(&m, h, 4);
    std::memcpy(&n, h + 8, 8);
    std::memcpy(&bs, h + 16, 4);
    std::memcpy(&nb, h + 20, 4);
    if (m != kGMagic || h[4] != 1 || h[5] || h[6] || h[7] || bs == 0 || div_up(n, bs) != nb ||
        jb.in_len < kGHdr + 8ull * (nb + 1ull)) {
      g.status = PIVCO_E_CORRUPT;
      continue;
    }
    if (n > jb.out_cap) { g.status = PIVCO_E_CAPACITY; continue; }
    g.n_total = n;
    g.n_blocks = nb;
    g.block_size = bs;
    blocks += nb;
    longest = std::max(longest, std::min<uint64_t>(n, bs));
  }
  // room for the batch's blocks, 8 bytes each, is part of the workspace that
  // callers were told to bring
  const uint64_t need = galign(count * sizeof(GJob) + 16, 256) + galign(8 * blocks + 16, 256);
  if (ws_bytes < need) return PIVCO_E_CAPACITY;
  if (count == 0) return PIVCO_OK;
  if (blocks > 0x7FFFFFFFull) return PIVCO_E_UNSUPPORTED;
  GJob *dj = static_cast<GJob *>(d_ws);
  if (count <= kGArgJobs) {
    GArgs a;
    std::copy(jobs.begin(), jobs.end(), a.j);
    hipLaunchKernelGGL(k_ginit, dim3(1), dim3(64), 0, s, dj, count, d_status, a);
  } else {
    if (hipMemcpyAsync(dj, jobs.data(), count * sizeof(GJob), hipMemcpyHostToDevice, s) != hipSuccess)
      return PIVCO_E_DEVICE;
    hipLaunchKernelGGL(k_gstatus, dim3((count + 255) / 256), dim3(256), 0, s, dj, count, d_status);
  }
  if (blocks) {
    const bool wide = blocks <= kGFew && longest > kGNarrow;
    hipLaunchKernelGGL(wide ? k_gdecode<1024> : k_gdecode<512>, dim3(static_cast<uint32_t>(blocks)),
                       dim3(wide ? 1024 : 512), 0, s, dj, count, static_cast<uint32_t>(blocks), d_status);
  }
  if (hipGetLastError() != hipSuccess) return PIVCO_E_DEVICE;
  if (hipStreamSynchronize(s) != hipSuccess) return PIVCO_E_DEVICE;
  return PIVCO_OK;
}

}  // extern "C"
