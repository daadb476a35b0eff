// Internal interface between the C ABI (fa_api.hip) and the kernel files.
#pragma once
#include "fa_common.h"

namespace fa {

struct FwdArgs {
  Problem p;
  const __bf16* Q;
  const __bf16* K;
  const __bf16* V;
  __bf16* O;
  float* LSE;
  // key sequence split over workgroups (0: not split): partial O [nsplit, tokens, Hq, d] and
  // partial logsumexp [nsplit] x (layout of LSE), float32, in caller-provided workspace
  int nsplit;
  float* Opart;
  float* Lpart;
  // key/value cache (split kernel only): sequence s attends to its first seqlens_k[s] keys (nullptr: all
  // p.Nk; values are clamped into 0 .. p.Nk). With a block table (nullptr: one slab of p.Nk rows per
  // sequence) K and V are pools of pages of 2^page_log2 rows (a multiple of 64) and key c of sequence s
  // is row c mod 2^page_log2 of page block_table[s * table_stride + (c >> page_log2)].
  const int32_t* seqlens_k;
  const int32_t* block_table;
  int page_log2, table_stride;
};

// Keys of sequence s in a cache with lengths of its own (a.seqlens_k is set).
__device__ __forceinline__ int cache_length(const FwdArgs& a, int s) {
  const int len = a.seqlens_k[s];
  return len < 0 ? 0 : (len < a.p.Nk ? len : a.p.Nk);
}

// Sequences of uneven cache lengths are handed out longest first: the workgroups of an XCD take
// their (sequence, head) pairs in launch order, and a long sequence that starts last leaves the
// other compute units idle at the end. The sequence index of the launch order is therefore read as a
// RANK, and the sequence of that rank (by length, ties by index) is found here: lane c counts the
// sequences that come before candidate c. Done by every wavefront for itself, from one load of all lengths whose lanes
// are then read in turn (a scalar load per sequence instead, each waited for, makes a chain of them before the first request
// of a key); batches of more than kRankMax sequences keep the launch order.
constexpr int kRankMax = 128;
struct CacheSequence {
  int s, len;  // the sequence, and its number of keys
};
__device__ __forceinline__ CacheSequence cache_sequence(const FwdArgs& a, int rank) {
  const int nseq = a.p.nseq, lane = threadIdx.x & 63;
  if (!a.seqlens_k) return {rank, a.p.Nk};
  if (nseq <= 1 || nseq > kRankMax) return {rank, cache_length(a, rank)};
  static_assert(kRankMax == 128, "two candidates per lane, and seven bits of an index in a key");
  const int c0 = lane, c1 = 64 + lane;
  const int len0 = cache_length(a, c0 < nseq ? c0 : 0), len1 = nseq > 64 ? cache_length(a, c1 < nseq ? c1 : 0) : 0;
  // (all keys differ, and a larger one goes first; where a length outgrows 25 bits the order is another one, but still an
  // order. Lanes without a sequence hold 0, which is larger than none.)
  const unsigned key0 = c0 < nseq ? ((unsigned)len0 << 7) | (unsigned)(127 - c0) : 0u;
  const unsigned key1 = c1 < nseq ? ((unsigned)len1 << 7) | (unsigned)(127 - c1) : 0u;
  int before0 = 0, before1 = 0;
  const int n0 = nseq < 64 ? nseq : 64;
  for (int j = 0; j < n0; j += 4) {
    unsigned k[4];
    for (int u = 0; u < 4; ++u) k[u] = (unsigned)__builtin_amdgcn_readlane((int)key0, j + u);
    for (int u = 0; u < 4; ++u) before0 += k[u] > key0 ? 1 : 0;
    if (nseq > 64)
      for (int u = 0; u < 4; ++u) before1 += k[u] > key1 ? 1 : 0;
  }
  for (int j = 0; j < nseq - 64; j += 4) {
    unsigned k[4];
    for (int u = 0; u < 4; ++u) k[u] = (unsigned)__builtin_amdgcn_readlane((int)key1, j + u);
    for (int u = 0; u < 4; ++u) before0 += k[u] > key0 ? 1 : 0;
    for (int u = 0; u < 4; ++u) before1 += k[u] > key1 ? 1 : 0;
  }
  const unsigned long long hit0 = __builtin_amdgcn_ballot_w64(c0 < nseq && before0 == rank);
  const unsigned long long hit1 = __builtin_amdgcn_ballot_w64(c1 < nseq && before1 == rank);
  const int l = hit0 ? __builtin_ctzll(hit0) : (hit1 ? __builtin_ctzll(hit1) : 0);
  return {hit0 ? l : 64 + l, __builtin_amdgcn_readlane(hit0 ? len0 : len1, l)};
}

// Shares of the row-block split kernel, in blocks of 64 keys: a sequence of `ncol` blocks is cut into at
// most nsplit equal shares, the same number for every length (shares of one size, of which a short
// sequence gets fewer, measured 5-15% slower at two shares: longest-first order then no longer goes by
// the work of a share), but not into shares of under kSplitMinBlocks blocks unless those of a full cache
// (cap_blocks) are that short: their start-up and partial results cost more than they even out. A
// sequence of one share needs no merge: the split kernel writes its O and LSE and fwd_merge_kernel passes
// its rows over.
constexpr int kSplitMinBlocks = 16;
__host__ __device__ inline int split_share_blocks(int ncol, int cap_blocks, int nsplit) {
  const int per = (ncol + nsplit - 1) / nsplit, full = (cap_blocks + nsplit - 1) / nsplit;
  const int least = full < kSplitMinBlocks ? full : kSplitMinBlocks;
  return per < least ? least : per;
}

struct BwdArgs {
  Problem p;
  const __bf16* Q;
  const __bf16* K;
  const __bf16* V;
  const __bf16* O;
  const __bf16* dO;
  const float* LSE;
  __bf16* dQ;
  __bf16* dK;
  __bf16* dV;
  float* Dvec;   // workspace: rowsum(dO o O), laid out like LSE
  // shares of the blocks of keys (key_shares in fa_bwd.hip): how many, and where their sums of dK, dV go, float32 [share][dK, dV][row of
  // K][p.d], key_rows rows of K; partial = nullptr: no room, not taken
  int shares, share_turn;  // (by how many XCDs a share's blocks are turned against those of the share before it)
  float* partial;
  long key_rows;
  bool keep_d;   // whoever asked for all three stages may run single ones on the same workspace: D has to be left there
  // gradient of the elementwise mask (mask instantiation of the dQ kernel only; nullptr: not asked for):
  // dM = dS in the element type, entry (s, h, r, c) at dM[s * dm_bs + h * dm_hs + r * dm_rs + c]
  __bf16* dM;
  long dm_bs, dm_hs, dm_rs;
};

// Room for the sums of the largest number of shares that key_shares takes, in rows of K (dK and dV make two of each); 0 where it takes
// none. nq: query rows of a sequence, or an upper bound.
constexpr long kShareRows = 65536;
constexpr int kMostShares = 16;
inline long share_rows(long key_rows, int Hq, int Hkv, long nq) {
  const long rows = key_rows * Hkv, group = Hkv > 0 ? Hq / Hkv : 0;
  if (group < 4 || group * nq <= (group < 8 ? 4800 : 2560) || rows <= 0 || 2 * rows > kShareRows) return 0;
  const long most = kShareRows / rows;
  return rows * (most < kMostShares ? most : kMostShares);
}

// FP8 (E4M3) forward: Q, K one byte per element in the token-major layout, V key-major
// [B, Hkv, d, vt_stride]; p.scale is the softmax scaling times the scales of Q and K
struct Fp8Args {
  Problem p;
  const void* Q;
  const void* K;
  const void* Vt;
  __bf16* O;
  float* LSE;
  long vt_stride;   // bytes between the rows of V^T: a multiple of 64, at least Nk rounded up to 64
  float descale_v;
};

hipError_t launch_fwd(const FwdArgs& a, int d, int causal, hipStream_t st);
// forward in workgroups of four wavefronts for grids that leave wavefront slots empty (fa_stream.hip); d in {64, 128}
hipError_t launch_fwd_stream(const FwdArgs& a, int d, int causal, hipStream_t st);
// the whole backward of short sequences as one kernel (fa_short.hip): d = 64, no options; whether a problem takes it
bool bwd_short_form(const Problem& p, int causal);
hipError_t launch_bwd_short(const BwdArgs& a, int causal, hipStream_t st);
// split forward for at most 32 (query row, head of the group) pairs per key/value head (fa_decode.hip):
// writes the shares' partial results like the split kernel; d in {64, 128}
hipError_t launch_fwd_decode(const FwdArgs& a, int d, int causal, hipStream_t st);
hipError_t launch_fwd_fp8(const Fp8Args& a, int d, int causal, hipStream_t st);
// stages: bit 0 D pre-pass, bit 1 dK/dV kernel, bit 2 dQ kernel
hipError_t launch_bwd(const BwdArgs& a, int d, int causal, int stages, hipStream_t st);
// ragged batches with two lengths: O (or dQ) = 0 and L = -inf for the query rows of sequences without keys
hipError_t launch_keyless_rows(const Problem& p, __bf16* out, float* lse, hipStream_t st);
// head dimension 256 (fa_d256.hip): plain problems only (no split, dropout, mask)
hipError_t launch_fwd256(const FwdArgs& a, int causal, hipStream_t st);
hipError_t launch_bwd256(const BwdArgs& a, int causal, int stages, hipStream_t st);
// register-resident MFMA loop: sink gets workgroups * 512 floats, clocks two counters
hipError_t launch_mfma_probe(float* sink, long long* clocks, int workgroups, int iters, int random_operands,
                             hipStream_t st);

}  // namespace fa
