// Shared device-side helpers for the gfx950 attention kernels: vector types,
// MFMA wrappers and the lane layouts they imply.
#pragma once
#include <hip/hip_runtime.h>
#include <stdint.h>

#include <type_traits>
#include <utility>

namespace fa {

typedef __attribute__((ext_vector_type(8))) __bf16 bf16x8;
typedef __attribute__((ext_vector_type(2))) __bf16 bf16x2;
typedef __attribute__((ext_vector_type(4))) short s16x4;
typedef __attribute__((ext_vector_type(8))) short s16x8;
typedef __attribute__((ext_vector_type(2))) float f32x2;
typedef __attribute__((ext_vector_type(4))) float f32x4;
typedef __attribute__((ext_vector_type(16))) float f32x16;
typedef __attribute__((ext_vector_type(4))) uint32_t u32x4;
typedef __attribute__((ext_vector_type(2))) uint32_t u32x2;

constexpr float kLog2e = 1.4426950408889634f;
constexpr float kLn2 = 0.6931471805599453f;

// Problem description shared by the forward and backward kernels. A "sequence"
// is one batch entry (dense) or one entry of cu_seqlens (packed ragged). A sequence has
// nq query rows and nk key/value rows (equal except through the two-length entry points);
// under the causal mask query r stands at position r + nk - nq of the keys.
struct Problem {
  const int32_t* cu_seqlens;  // device, nseq + 1 entries; nullptr for the dense layout
  const int32_t* cu_seqlens_k;  // ragged with two lengths: the key/value rows' offsets; else nullptr
  int nseq;                   // number of sequences (dense: batch size)
  int N;                      // dense: number of query rows; ragged: upper bound on any length
  int Nk;                     // dense: number of key/value rows; ragged: same bound
  int Hq, Hkv, G;             // G = Hq / Hkv
  int d;                      // head dimension in memory (a multiple of 8); kernels pad it to 64 or 128 on chip
  int total_tokens;
  long lse_seq_stride;        // dense: Hq * N, ragged: 0
  long lse_head_stride;       // dense: N, ragged: total_tokens
  float scale;                // softmax scaling
  float scale_log2e;          // scale * log2(e)
  int f16;                    // element type of the 16-bit tensors: 0 bfloat16, 1 IEEE half precision
  // dropout on P (drop_thr = 0: none): an entry is kept when its byte of the hash is >= drop_thr
  uint32_t drop_thr;          // round(256 p), 1 .. 255
  uint32_t drop_seed;         // (seed mod 2^32) xor (seed >> 32) * 0x27D4EB2F
  float drop_rp, drop_log2;   // 1 / (1 - drop_thr / 256) and its base-2 logarithm
  // elementwise mask added to the scaled scores (nullptr: none): bfloat16, finite or -inf,
  // element (s, h, r, c) at mask[s * mask_bs + h * mask_hs + r * mask_rs + c]; a stride of 0
  // shares the mask over sequences or heads; mask_rs >= Nk rounded up to 8, a multiple of 8
  const __bf16* mask;
  long mask_bs, mask_hs, mask_rs;
  // sliding window (local attention): with query r at position q = r + nk - nq among the keys, key c
  // is visible iff q - win_left <= c <= q + win_right; a negative bound is no bound. Only read
  // by the LOCAL instantiations (the entry points send "no bound at all" and "win_right = 0
  // alone" to the plain and the causal kernels).
  int win_left, win_right;
  // block-sparse pattern (nullptr: none; LOCAL instantiations only): one byte per block of
  // 2^bmask_log2 x 2^bmask_log2 entries of S (a power of two, at least 64), row blocks counted
  // from query 0 and key blocks from key 0; byte (s, h, rb, cb) at
  // bmask[s * bmask_bs + h * bmask_hs + rb * bmask_cols + cb], 0 = the block is removed;
  // a stride of 0 shares the pattern over sequences or heads
  const uint8_t* bmask;
  long bmask_bs, bmask_hs;
  int bmask_cols, bmask_log2;
};
// the LOCAL template parameter of the kernels: nothing, a sliding window, a block-sparse pattern (perhaps with a window)
constexpr int kNoPattern = 0, kWindow = 1, kBlocks = 2;
constexpr int kPatternWords = 64;  // 64-bit words of a wavefront's activity bitmap in LDS: 4096 blocks or tiles

struct SeqInfo {
  long tok0;   // first query row of the sequence in the packed [tokens, H, d] view
  long tok0k;  // first key/value row
  int n;       // query rows
  int nk;      // key/value rows
};

__device__ __forceinline__ SeqInfo seq_info(const Problem& p, int s) {
  SeqInfo r;
  if (p.cu_seqlens) {
    int a = p.cu_seqlens[s];
    r.tok0 = r.tok0k = a;
    r.n = r.nk = p.cu_seqlens[s + 1] - a;
    if (p.cu_seqlens_k) {
      a = p.cu_seqlens_k[s];
      r.tok0k = a;
      r.nk = p.cu_seqlens_k[s + 1] - a;
    }
  } else {
    r.tok0 = (long)s * p.N;
    r.tok0k = (long)s * p.Nk;
    r.n = p.N;
    r.nk = p.Nk;
  }
  return r;
}

// Launch index -> (block of rows or columns, head, sequence).
//
// The chip has 8 XCDs, each with 32 CUs and a private 4 MiB L2; the hardware hands
// consecutive workgroup indices to consecutive XCDs. Every workgroup of one (head,
// sequence) pair streams the same K/V (or Q/dO) through L2, about 4 MiB at d = 128 and
// N = 8192. The mapping below therefore gives all blocks of a pair to ONE XCD and lets an
// XCD walk its pairs one after the other, so its 32 CUs share one pair's operands at a time
// instead of thrashing L2 with eight. Under the causal mask block costs differ by up to
// the number of blocks, so there the XCD's pairs are interleaved and all their heaviest
// blocks are dispatched first (longest-processing-time order), lightest last.
// Pairs that do not make up a full set of eight leave XCDs without work (one head of a long sequence: seven of them).
// Where an XCD that has one pair more than another would have more blocks than fit on it at once (Place::slots), the blocks of the pairs past the last full set, up to seven pairs' worth, are dealt to all XCDs in turn (`spread_pairs`;
// MI355X, us: a cache of 10 pairs, 5 x 416 new queries on up to 14848 keys, 2 heads of 128: 69.9 -> 43.4; forward and backward of 25
// packed sequences of up to 4067, 2 heads of 128: 434 -> 391, of 27 x 832, 4 heads of 128: 213 -> 206). Where all of
// them fit they stay where they were: 1 x 5056, 2 heads of 64, spread over eight L2s took 62.7 instead of 61.2.
// Kernels are launched on grid_size(nblk, pairs) workgroups; indices that fall past the last block return valid = false.
constexpr int kXcds = 8, kXcdUnits = 32;  // compute units of an XCD
struct BlockCoord {
  int blk, head, seq;
  bool valid;
};
// A workgroup's place among those of its kind (the grid, or a part of it that begins at a multiple of kXcds), and how many
// of them an XCD holds at once (beside those of another kind).
struct Place {
  unsigned index;
  int slots;
};
__host__ __device__ inline int spread_pairs(int nblk, int pairs, int slots) {
  return (pairs + kXcds - 1) / kXcds * nblk > slots ? pairs % kXcds : 0;
}
__host__ __device__ inline unsigned grid_size(int nblk, int pairs, int slots) {
  const int rest = spread_pairs(nblk, pairs, slots);
  return (unsigned)(kXcds * ((pairs - rest + kXcds - 1) / kXcds * nblk + (rest * nblk + kXcds - 1) / kXcds));
}
// Packed batches (ragged_coord): the real blocks of all pairs are numbered through, or of the pairs of each XCD, of
// which one may then have a pair more than another.
__host__ __device__ inline bool packed_through(int nblk, int pairs, int slots) {
  return pairs < 64 && spread_pairs(nblk, pairs, slots) != 0;
}
// The grid of a kernel that goes by row_block_coord (heads: p.Hq) or key_block_coord (p.Hkv)
inline unsigned grid_size(const Problem& p, int nblk, int heads, int slots) {
  const int pairs = heads * p.nseq;
  if (!p.cu_seqlens || packed_through(nblk, pairs, slots)) return grid_size(nblk, pairs, slots);
  return (unsigned)((pairs + kXcds - 1) / kXcds * kXcds * nblk);
}
// `group` > 1 (kernels whose grid runs over QUERY heads that share key/value heads in groups of
// that size): heads are handed out so that the heads of one group follow each other at a
// distance of nheads / group pairs. With a multiple of 8 key/value heads they then land on the
// same XCD, whose L2 holds the group's K and V once instead of every XCD holding them all.
// BACK: the pairs from the last to the first (see launch_bwd_d).
template <bool WORK_SORTED, bool BACK = false>
__device__ __forceinline__ BlockCoord block_coord(Place at, int nblk, int nheads, int nseq, int group = 1) {
  const int x = at.index % kXcds, k = at.index / kXcds;
  const int pairs = nheads * nseq, rest = spread_pairs(nblk, pairs, at.slots);
  const int own = (pairs - rest + kXcds - 1) / kXcds;  // pairs that one XCD has to itself
  BlockCoord c;
  int pl;  // which of them
  if (WORK_SORTED) {  // causal: the XCD's pairs take turns, every pair's heaviest blocks first
    c.blk = rest ? kXcds * k / pairs : k / own;
    pl = k - c.blk * own;
  } else {  // one pair at a time
    pl = k / nblk;
    c.blk = k - pl * nblk;
  }
  int pr = (BACK ? own - 1 - pl : pl) * kXcds + x;
  if (rest) {
    if (WORK_SORTED) {
      // Block b of the q-th spread pair goes to XCD (rest * b + q) % 8. before(b): blocks of this XCD that come before those with
      // index b.
      auto before = [&](int b) { return own * b + (rest * b + kXcds - 1 - x) / kXcds; };
      while (before(c.blk + 1) <= k) ++c.blk;
      while (before(c.blk) > k) --c.blk;
      pl = k - before(c.blk);
      pr = pl < own ? (BACK ? own - 1 - pl : pl) * kXcds + x : own * kXcds + ((x - rest * c.blk) & (kXcds - 1));
    } else if (pl >= own) {
      const int i = (k - own * nblk) * kXcds + x;
      pr = own * kXcds + i / nblk;
      c.blk = i % nblk;
    }
  }
  c.seq = pr / nheads;
  c.head = pr - c.seq * nheads;
  if (group > 1) {  // (a branch: a division is a chain of some twenty instructions in front of the first request)
    const int nkv = nheads / group, in = c.head / nkv;
    c.head = (c.head - in * nkv) * group + in;
  }
  c.valid = pr < pairs && c.blk < nblk;
  return c;
}

// Sum over the 64 lanes of a wavefront (all active), the same value in every lane.
__device__ __forceinline__ int wave_sum(int x) {
  x += __builtin_amdgcn_update_dpp(0, x, 0x111, 0xf, 0xf, true);  // row_shr 1, 2, 4, 8: lane 15 of a row has its sum
  x += __builtin_amdgcn_update_dpp(0, x, 0x112, 0xf, 0xf, true);
  x += __builtin_amdgcn_update_dpp(0, x, 0x114, 0xf, 0xf, true);
  x += __builtin_amdgcn_update_dpp(0, x, 0x118, 0xf, 0xf, true);
  x += __builtin_amdgcn_update_dpp(0, x, 0x142, 0xa, 0xf, false);  // row_bcast 15, then 31
  x += __builtin_amdgcn_update_dpp(0, x, 0x143, 0xc, 0xf, false);
  return __builtin_amdgcn_readlane(x, 63);
}

// Launch index -> work of a packed ragged batch. The grid has room for the longest possible sequence in
// every (head, sequence) pair, so most launch indices of block_coord's numbering stand for blocks that
// a shorter sequence does not have. Such a workgroup is gone at once, but the dispatcher deals
// workgroups to the shader engines in turn and in order: empty ones between real ones leave some
// engines with fewer real workgroups than others, and compute units idle. The real blocks are therefore
// numbered without gaps, the empty indices all behind them, heaviest blocks first:
//  * LEVELS (causal): a block's work is what remains of its sequence from there on, `left` blocks
//    (1 .. blocks of the sequence); all blocks with the most left first, pair by pair, and so on down.
//  * else: every block of a sequence costs the same; the pairs with the most blocks first, block by block.
// 16 sequences of 758 .. 3951 tokens (37954 in all), 32 heads on 8, d = 128, causal: the dK/dV kernel takes
// 2.05 ms with the gaps and 1.57 ms without (the pass of three kernels 4.26 -> 3.82 ms).
// Lane l holds the number of blocks of the pairs l, l + 64, .. of this XCD (or of all: packed_through); the number of real blocks
// with at least `left` left (the number of blocks of pairs with at least that many) falls with `left`, and
// a binary search finds where launch index k stands. Up to 64 * kRaggedChunks pairs per XCD; beyond (and for
// dense batches, which have no gaps) block_coord's order stays.
constexpr int kRaggedChunks = 4;
struct RaggedCoord {
  int blocks, left, blk, head, seq;  // of the pair; LEVELS: left, else blk (counted from the front)
  bool valid;
};
template <bool LEVELS>
__device__ __forceinline__ RaggedCoord ragged_coord(Place at, const int32_t* cu, int rows, int nblk, int nheads, int nseq,
                                                    int group) {
  const int lane = __builtin_amdgcn_mbcnt_hi(~0u, __builtin_amdgcn_mbcnt_lo(~0u, 0u));
  const int pairs = nheads * nseq, lists = packed_through(nblk, pairs, at.slots) ? 1 : kXcds;  // (a list per XCD, or one for all)
  const int x = at.index % lists, k = at.index / lists;
  const int chunks = ((pairs + lists - 1) / lists + 63) / 64;
  int nb[kRaggedChunks];
#pragma unroll
  for (int c = 0; c < kRaggedChunks; ++c) {
    nb[c] = 0;
    const int pr = (64 * c + lane) * lists + x;
    if (c < chunks && pr < pairs) {
      const int s = pr / nheads;
      const int b = (cu[s + 1] - cu[s] + rows - 1) / rows;
      nb[c] = b < 0 ? 0 : (b < nblk ? b : nblk);
    }
  }
  auto ahead = [&](int v) {  // real blocks with at least v left (blocks of pairs with at least v)
    int t = 0;
#pragma unroll
    for (int c = 0; c < kRaggedChunks; ++c) t += nb[c] < v ? 0 : (LEVELS ? nb[c] - v + 1 : nb[c]);
    return wave_sum(t);
  };
  RaggedCoord r = {0, 0, 0, 0, 0, false};
  if (ahead(1) <= k) return r;
  int lo = 1, hi = nblk;  // the largest v with ahead(v) > k
  while (lo < hi) {
    const int mid = (lo + hi + 1) >> 1;
    if (ahead(mid) > k) lo = mid;
    else hi = mid - 1;
  }
  const int nth = k - ahead(lo + 1);
  int which = LEVELS ? nth : nth / lo;  // which of the pairs with that many left (exactly that many blocks)
  int pl = 0;
#pragma unroll
  for (int c = 0; c < kRaggedChunks; ++c) {
    const bool on = LEVELS ? nb[c] >= lo : nb[c] == lo;
    const unsigned long long m = __builtin_amdgcn_ballot_w64(on);
    const int before = __builtin_amdgcn_mbcnt_hi((unsigned)(m >> 32), __builtin_amdgcn_mbcnt_lo((unsigned)m, 0u));
    const unsigned long long hit = __builtin_amdgcn_ballot_w64(on && before == which);
    if (hit) {
      const int l = __builtin_ctzll(hit);
      pl = 64 * c + l;
      r.blocks = __builtin_amdgcn_readlane(nb[c], l);
    }
    which -= __builtin_popcountll(m);
  }
  const int pr = pl * lists + x, hp = pr % nheads, nkv = nheads / group;
  r.left = lo;
  r.blk = LEVELS ? 0 : nth % lo;
  r.head = (hp % nkv) * group + hp / nkv;  // (as in block_coord)
  r.seq = pr / nheads;
  r.valid = true;
  return r;
}
__device__ __forceinline__ bool ragged_order(int pairs) { return pairs <= kXcds * 64 * kRaggedChunks; }

// (through the first lane: the compiler would keep the coordinates, and all that follows from them, per lane)
__device__ __forceinline__ BlockCoord scalar_coord(BlockCoord c) {
  const int b = __builtin_amdgcn_readfirstlane(c.valid ? c.blk : -1);
  return {b, __builtin_amdgcn_readfirstlane(c.head), __builtin_amdgcn_readfirstlane(c.seq), b >= 0};
}

// Which block of `rows` query rows (heaviest first) of which query head a workgroup takes; blk counts from row 0.
// RAGGED (p.cu_seqlens is set) is a parameter of the instantiation, not asked here: short dense batches, whose time is
// the chain of one workgroup, feel the search even as code that they jump over.
template <bool CAUSAL, bool RAGGED, bool BACK = false>
__device__ __forceinline__ BlockCoord row_block_coord(Place at, const Problem& p, int rows) {
  const int nblk = (p.N + rows - 1) / rows;
  if (RAGGED && ragged_order(p.Hq * p.nseq)) {
    const RaggedCoord r = ragged_coord<CAUSAL>(at, p.cu_seqlens, rows, nblk, p.Hq, p.nseq, p.G);
    return scalar_coord({CAUSAL ? r.left - 1 : r.blk, r.head, r.seq, r.valid});
  }
  BlockCoord c = block_coord<CAUSAL, BACK>(at, nblk, p.Hq, p.nseq, p.G);
  c.blk = nblk - 1 - c.blk;
  return c;
}
// Which block of `keys` keys of which key/value head; blk counts from key 0, under the causal rule the
// heaviest block. A block's work then grows with the number of rows below it, not with its index: in
// block_coord's order (batches with very many pairs) block indices therefore count from the END of the
// longest possible sequence, and the blocks that a shorter one does not have are not valid.
template <bool CAUSAL, bool RAGGED>
__device__ __forceinline__ BlockCoord key_block_coord(Place at, const Problem& p, int keys) {
  const int nblk = (p.Nk + keys - 1) / keys;
  if (RAGGED && ragged_order(p.Hkv * p.nseq)) {
    const RaggedCoord r =
        ragged_coord<CAUSAL>(at, p.cu_seqlens_k ? p.cu_seqlens_k : p.cu_seqlens, keys, nblk, p.Hkv, p.nseq, 1);
    return scalar_coord({CAUSAL ? r.blocks - r.left : r.blk, r.head, r.seq, r.valid});
  }
  BlockCoord c = block_coord<CAUSAL>(at, nblk, p.Hkv, p.nseq);
  if (CAUSAL && RAGGED && c.valid) {
    c.blk -= nblk - (seq_info(p, c.seq).nk + keys - 1) / keys;
    c.valid = c.blk >= 0;
  }
  return c;
}

// D = A(32 x 16) * B(16 x 32) + C on one wavefront, 16-bit inputs, fp32 accumulate.
// Lane l supplies A[l % 32][8 * (l / 32) + t] and B[8 * (l / 32) + t][l % 32], t = 0..7,
// and owns C[8 * (r / 4) + 4 * (l / 32) + (r % 4)][l % 32] in register r = 0..15.
// The kernels move 16-bit elements around as raw bits (bf16x8 is just 128 bits of them);
// the element type only matters here, where they are multiplied, and in pack2 below, where
// float32 results are rounded: F16 = false means bfloat16, F16 = true IEEE half precision.
typedef __attribute__((ext_vector_type(8))) _Float16 f16x8;
typedef __attribute__((ext_vector_type(2))) _Float16 f16x2;
template <bool F16 = false>
__device__ __forceinline__ f32x16 mfma32(bf16x8 a, bf16x8 b, f32x16 c) {
  if constexpr (F16)
    return __builtin_amdgcn_mfma_f32_32x32x16_f16(__builtin_bit_cast(f16x8, a), __builtin_bit_cast(f16x8, b), c, 0, 0, 0);
  else
    return __builtin_amdgcn_mfma_f32_32x32x16_bf16(a, b, c, 0, 0, 0);
}

// The same product with the registers of its accumulator and of B chosen by hand, for kernels of one wavefront per SIMD:
// the 512 registers of a wavefront are two files of 256, vector and accumulation registers (VGPR, AGPR); an MFMA takes its
// accumulator from either and vector instructions only see the first. Left to itself the compiler keeps EVERY
// accumulator in the second and copies scores back and forth for the softmax, or moves the long-lived accumulators
// from one file to the other around every branch (d = 256 dQ kernel: 432 register copies beside 96 MFMAs).
//   mfma32_agpr     C in AGPRs, B in VGPRs            mfma32_vgpr_ab  C in VGPRs, B in AGPRs
//   mfma32_vgpr     C in VGPRs, B in VGPRs            (FIRST: C starts from zero)
// Inline assembly is opaque to the compiler's hazard recogniser, so the callers keep the rules: two wait states between a
// vector instruction that writes an operand and the MFMA, and settled() between the last MFMA on an accumulator and a
// vector instruction that touches it, unless two other MFMAs lie between (tests/test_kernel_resources.py walks
// the compiler's output for both).
template <bool F16>
__device__ __forceinline__ void mfma32_agpr(f32x16& c, bf16x8 a, bf16x8 b) {
  if constexpr (F16) asm volatile("v_mfma_f32_32x32x16_f16 %0, %1, %2, %0" : "+a"(c) : "v"(a), "v"(b));
  else asm volatile("v_mfma_f32_32x32x16_bf16 %0, %1, %2, %0" : "+a"(c) : "v"(a), "v"(b));
}
template <bool F16, bool FIRST>
__device__ __forceinline__ void mfma32_vgpr_ab(f32x16& c, bf16x8 a, bf16x8 b) {
  if constexpr (F16 && FIRST) asm volatile("v_mfma_f32_32x32x16_f16 %0, %1, %2, 0" : "=&v"(c) : "v"(a), "a"(b));
  else if constexpr (F16) asm volatile("v_mfma_f32_32x32x16_f16 %0, %1, %2, %0" : "+v"(c) : "v"(a), "a"(b));
  else if constexpr (FIRST) asm volatile("v_mfma_f32_32x32x16_bf16 %0, %1, %2, 0" : "=&v"(c) : "v"(a), "a"(b));
  else asm volatile("v_mfma_f32_32x32x16_bf16 %0, %1, %2, %0" : "+v"(c) : "v"(a), "a"(b));
}
template <bool F16, bool FIRST>
__device__ __forceinline__ void mfma32_vgpr(f32x16& c, bf16x8 a, bf16x8 b) {
  if constexpr (F16 && FIRST) asm volatile("v_mfma_f32_32x32x16_f16 %0, %1, %2, 0" : "=&v"(c) : "v"(a), "v"(b));
  else if constexpr (F16) asm volatile("v_mfma_f32_32x32x16_f16 %0, %1, %2, %0" : "+v"(c) : "v"(a), "v"(b));
  else if constexpr (FIRST) asm volatile("v_mfma_f32_32x32x16_bf16 %0, %1, %2, 0" : "=&v"(c) : "v"(a), "v"(b));
  else asm volatile("v_mfma_f32_32x32x16_bf16 %0, %1, %2, %0" : "+v"(c) : "v"(a), "v"(b));
}
// (an MFMA of 8 passes needs 12 wait states before its result may be touched)
__device__ __forceinline__ void settled(f32x16& a) { asm volatile("s_nop 15" : "+v"(a)); }
__device__ __forceinline__ void settled(f32x16& a, f32x16& b) { asm volatile("s_nop 15" : "+v"(a), "+v"(b)); }
template <int N>
__device__ __forceinline__ void settled(f32x16 (&c)[N]) {
  if constexpr (N == 2) asm volatile("s_nop 15" : "+v"(c[0]), "+v"(c[1]));
  else asm volatile("s_nop 15" : "+v"(c[0]), "+v"(c[1]), "+v"(c[2]), "+v"(c[3]));
}
// (as operands of ONE statement: a copy of an accumulator that the compiler makes then stands on the right side of the wait)
__device__ __forceinline__ void agpr_settled(f32x16 (&c)[8]) {
  asm volatile("s_nop 15" : "+a"(c[0]), "+a"(c[1]), "+a"(c[2]), "+a"(c[3]), "+a"(c[4]), "+a"(c[5]), "+a"(c[6]), "+a"(c[7]));
}
// Before a stream of MFMAs: the accumulators are in the registers that it uses.
__device__ __forceinline__ void agpr_ready(f32x16 (&c)[8]) {
  asm volatile("s_nop 1" : "+a"(c[0]), "+a"(c[1]), "+a"(c[2]), "+a"(c[3]), "+a"(c[4]), "+a"(c[5]), "+a"(c[6]), "+a"(c[7]));
}

// f(integral_constant<int, 0>) .. f(integral_constant<int, N - 1>): loops that have to be unrolled whatever their size
template <class F, int... I>
__device__ __forceinline__ void static_for_each(F f, std::integer_sequence<int, I...>) {
  (f(std::integral_constant<int, I>{}), ...);
}
template <int N, class F>
__device__ __forceinline__ void static_for(F f) {
  static_for_each(f, std::make_integer_sequence<int, N>{});
}

// Row of the 32 x 32 accumulator tile that register r of lane-half hh holds.
__device__ __forceinline__ constexpr int acc_row(int r, int hh) { return 8 * (r / 4) + 4 * hh + (r % 4); }

typedef __attribute__((address_space(3))) s16x4 lds_s16x4;

// Transposing LDS read (ds_read_b64_tr_b16). Within each group of 16 lanes,
// lane p passes the address of 4 consecutive 16-bit elements; lane i receives,
// in slot t, element (i % 4) of the four that lane (i / 4 + 4 * t) pointed at.
__device__ __forceinline__ s16x4 lds_read_tr(const __bf16* ptr) {
  return __builtin_amdgcn_ds_read_tr16_b64_v4i16((lds_s16x4*)ptr);
}

// Maximum / sum of a value with the one held by lane l ^ 32 (v_permlane32_swap).
__device__ __forceinline__ float max_with_partner32(float x) {
  int xi = __builtin_bit_cast(int, x);
  auto sw = __builtin_amdgcn_permlane32_swap(xi, xi, false, false);
  return fmaxf(__builtin_bit_cast(float, (int)sw[0]), __builtin_bit_cast(float, (int)sw[1]));
}

__device__ __forceinline__ float max3(float a, float b, float c) { return __builtin_fmaxf(__builtin_fmaxf(a, b), c); }
// Largest score of this lane's row in a block of 64 keys (S^T: two accumulators of 32 keys, the row's other half in the partner lane).
__device__ __forceinline__ float row_maximum(const f32x16 (&S)[2]) {
  float mx = max3(S[0][0], S[0][1], S[1][0]);
#pragma unroll
  for (int r = 2; r < 16; r += 2) mx = max3(mx, S[0][r], S[0][r + 1]);
  mx = max3(mx, S[1][1], S[1][2]);
  mx = fmaxf(mx, S[1][3]);
#pragma unroll
  for (int r = 4; r < 16; r += 2) mx = max3(mx, S[1][r], S[1][r + 1]);
  return max_with_partner32(mx);
}
// The reference of the running softmax is only advanced (and O, l rescaled) when a lane's share
// of a block's row sum exceeds 2^kLazyLog2 (instantiations without the fast path: when some
// row's maximum outgrew the reference by that factor); until then exponentials are taken against
// the older reference and may reach 2^kLazyLog2. Half precision operands end at 65504 = 2^16;
// bfloat16 has float32's range, and the wider margin saves most of the remaining advances when the
// scores spread widely (3x the usual range: the row maximum grows by some 20 bits over 16k keys).
// All 16-bit forward kernels go by these: the size of the grid chooses between forms whose results are the same bits.
template <bool F16>
constexpr int kLazyLog2 = F16 ? 8 : 20;
template <bool F16>
__device__ __forceinline__ bool reference_outgrown(float share) {
  return __builtin_amdgcn_ballot_w64(share > (float)(1 << kLazyLog2<F16>)) != 0;
}
// Keys of a block (row_maximum) past `lim`, the last one that the row sees, counted from this lane's first, leave the softmax.
__device__ __forceinline__ void mask_past(f32x16 (&S)[2], int lim) {
#pragma unroll
  for (int kt = 0; kt < 2; ++kt)
#pragma unroll
    for (int r = 0; r < 16; ++r) S[kt][r] = 32 * kt + acc_row(r, 0) > lim ? -INFINITY : S[kt][r];
}

__device__ __forceinline__ float sum_with_partner32(float x) {
  int xi = __builtin_bit_cast(int, x);
  auto sw = __builtin_amdgcn_permlane32_swap(xi, xi, false, false);
  return __builtin_bit_cast(float, (int)sw[0]) + __builtin_bit_cast(float, (int)sw[1]);
}

// Two float32 values rounded (to nearest even) to the 16-bit element type, packed low | high.
template <bool F16 = false>
__device__ __forceinline__ uint32_t pack2(float lo, float hi) {
  f32x2 v = {lo, hi};
  if constexpr (F16) {
    f16x2 r = __builtin_convertvector(v, f16x2);
    return __builtin_bit_cast(uint32_t, r);
  } else {
    bf16x2 r = __builtin_convertvector(v, bf16x2);
    return __builtin_bit_cast(uint32_t, r);
  }
}

// Registers 8s .. 8s+7 of an accumulator tile, rounded to the element type, as an MFMA operand.
template <bool F16 = false>
__device__ __forceinline__ bf16x8 pack8(const f32x16& v, int s) {
  u32x4 r;
  r[0] = pack2<F16>(v[8 * s + 0], v[8 * s + 1]);
  r[1] = pack2<F16>(v[8 * s + 2], v[8 * s + 3]);
  r[2] = pack2<F16>(v[8 * s + 4], v[8 * s + 5]);
  r[3] = pack2<F16>(v[8 * s + 6], v[8 * s + 7]);
  return __builtin_bit_cast(bf16x8, r);
}

__device__ __forceinline__ float fast_exp2(float x) { return __builtin_amdgcn_exp2f(x); }
__device__ __forceinline__ float fast_log2(float x) { return __builtin_amdgcn_logf(x); }

// The exponentials of a block (row_maximum) against the reference -nref, in the exponent's base, rounded into the operands
// of the second product, and this lane's two shares of the row sum.
template <bool F16>
__device__ __forceinline__ void block_exponentials(const f32x16 (&S)[2], float c2, float nref, bf16x8 (&P)[2][2], float& rs0, float& rs1) {
  rs0 = rs1 = 0.f;
#pragma unroll
  for (int kt = 0; kt < 2; ++kt) {
    f32x16 E;
#pragma unroll
    for (int r = 0; r < 16; r += 2) {
      E[r] = fast_exp2(__builtin_fmaf(S[kt][r], c2, nref));
      E[r + 1] = fast_exp2(__builtin_fmaf(S[kt][r + 1], c2, nref));
      rs0 += E[r];
      rs1 += E[r + 1];
    }
    P[kt][0] = pack8<F16>(E, 0);
    P[kt][1] = pack8<F16>(E, 1);
  }
}

// Element t of 8 raw 16-bit elements, widened to float32.
template <bool F16>
__device__ __forceinline__ float widen(bf16x8 v, int t) {
  if constexpr (F16) return (float)__builtin_bit_cast(f16x8, v)[t];
  else return (float)v[t];
}

// acc + the sum of the products of 8 raw 16-bit elements, one after the other. Every kernel that sums D = rowsum(dO o O) does it by
// this chain, so that D is the same bits whoever forms it. (Held step by step: the compiler would otherwise take two products of
// half precision together in some kernels, v_dot2c_f32_f16, and not in others.)
template <bool F16>
__device__ __forceinline__ float dot8(bf16x8 a, bf16x8 b, float acc) {
#pragma unroll
  for (int t = 0; t < 8; ++t) {
    acc = __builtin_fmaf(widen<F16>(a, t), widen<F16>(b, t), acc);
    if constexpr (F16) asm("" : "+v"(acc));
  }
  return acc;
}

// The 16-bit element in the low (hi = false) or high half of a 32-bit word, widened to float32.
template <bool F16>
__device__ __forceinline__ float widen_half(uint32_t w, bool hi) {
  if constexpr (F16) return (float)__builtin_bit_cast(_Float16, (unsigned short)(hi ? w >> 16 : w));
  else return __builtin_bit_cast(float, hi ? (w & 0xffff0000u) : (w << 16));
}

// Dropout generator (defined by this library, the same function as the CPU checker's): for
// head index bh = sequence * Hq + head, query r and key c,
//   x = (c / 4) * 0x9E3779B1 + r * 0x85EBCA77 + (seed_mix xor bh * 0xC2B2AE3D), mixed by
//   drop_mix; entry (r, c) is kept when byte c % 4 of x is >= the threshold.
constexpr uint32_t kDropCol = 0x9E3779B1u, kDropRow = 0x85EBCA77u, kDropHead = 0xC2B2AE3Du;
__device__ __forceinline__ uint32_t drop_mix(uint32_t x) {
  x ^= x >> 16;
  x *= 0x7FEB352Du;
  x ^= x >> 15;
  x *= 0x846CA68Bu;
  x ^= x >> 16;
  return x;
}

// The value that lane u of this lane's quad (four neighbouring lanes) holds; u is a constant after unrolling.
__device__ __forceinline__ uint32_t quad_lane(uint32_t x, int u) {
  switch (u) {
    case 0: return (uint32_t)__builtin_amdgcn_mov_dpp((int)x, 0x00, 0xf, 0xf, true);
    case 1: return (uint32_t)__builtin_amdgcn_mov_dpp((int)x, 0x55, 0xf, 0xf, true);
    case 2: return (uint32_t)__builtin_amdgcn_mov_dpp((int)x, 0xaa, 0xf, 0xf, true);
    default: return (uint32_t)__builtin_amdgcn_mov_dpp((int)x, 0xff, 0xf, 0xf, true);
  }
}

}  // namespace fa
