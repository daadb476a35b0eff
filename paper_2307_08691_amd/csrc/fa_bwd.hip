// Backward pass of exact attention for gfx950 (Algorithm 2 of the paper).
//
// (Short sequences at d = 64: one kernel, fa_short.hip.) Three parts; the two kernels stand in fa_bwd_work.h. The full backward is two
// launches on the caller's stream: the pre-pass, then the other two side by side in one grid (fa_bwd_joint.h), or, on grids that leave
// no compute units idle either way, the third, which then sums D itself (OWN_D), and the second. Where few blocks of keys stand
// for long chains, several workgroups share each and a merge follows (key_shares).
//   1. prep:  D = rowsum(dO o O) (Algorithm 2, line 4)
//   2. dK/dV: one workgroup per block of 256 keys of one (sequence, key/value head)
//             (section 3.2 "Backward pass"); it loops over the query heads that share the
//             key/value head and over the row blocks i, recomputes P from the saved
//             logsumexp (line 11) and keeps dK_j, dV_j in MFMA accumulators for the whole
//             loop (lines 12-16 without line 15)
//   3. dQ:    one workgroup per block of 256 query rows; it loops over the column blocks,
//             recomputes P and dS and keeps dQ_i in MFMA accumulators (line 15)
//
// The paper accumulates dQ from the column-block workers with atomic adds (section 3.2).
// On MI355X float32 atomics into L2 retire at roughly 1.3 TB/s chip-wide: with them the
// single-kernel form of Algorithm 2 spent more than half its time waiting for the atomic
// unit (6.8 ms against 3.1 ms with the atomics removed, d = 128, N = 8192, 32 heads). The
// dQ pass here instead recomputes S and dP (7 products instead of 5) and needs no
// cross-workgroup accumulation at all; dQ, dK and dV are bit-reproducible.
//
// Lane layouts. dK/dV kernel: scores are computed UN-transposed, S = Q_i K_j^T, so a lane
// holds one key column; P and dS, rounded to bf16, are directly the right-hand operands of
// dV_j^T += dO_i^T P and dK_j^T += Q_i^T dS (contractions over the query rows), whose
// left-hand operands come from transposing LDS reads of the row-major Q_i / dO_i tiles.
// dQ kernel: scores are computed transposed, S^T = K_j Q_i^T, so a lane holds one query
// row (L_i, D_i are per-lane scalars) and dS^T in bf16 is the right-hand operand of
// dQ_i^T += K_j^T dS^T, with K_j^T from transposing reads of the K tile.
#include "fa_bwd_work.h"
#include "fa_common.h"
#include "fa_kernels.h"
#include "fa_lds.h"

namespace fa {

__device__ __forceinline__ long stat_index(const Problem& p, long tok, int h) {
  // index of (token, head) in the [B, Hq, N] (dense) or [Hq, T] (ragged) statistics layout
  if (p.cu_seqlens) return (long)h * p.lse_head_stride + tok;
  long b = tok / p.N, r = tok - b * p.N;
  return b * p.lse_seq_stride + (long)h * p.lse_head_stride + r;
}

// D = rowsum(dO o O) (line 4) as the dQ kernel sums it: the same bits. Two lanes to a row, one for every other 16 bytes.
template <int D, bool F16>
__global__ __launch_bounds__(256) void bwd_prep_kernel(BwdArgs a) {
  constexpr int KS = D / 16, ROWB = 2 * D, STAGE = 32 * ROWB;
  __shared__ __attribute__((aligned(1024))) char smem[D == 256 ? 1 : 8 * STAGE];
  const int lane = threadIdx.x & 63, lq = lane & 31, hh = lane >> 5;
  const int w = __builtin_amdgcn_readfirstlane(threadIdx.x >> 6);
  const long nrows = (long)a.p.total_tokens * a.p.Hq;
  const long row0 = (long)blockIdx.x * kPrepRows + 32 * w, row = row0 + lq;
  if (row0 >= nrows) return;
  const int dh = a.p.d;  // row length in memory, at most D
  bf16x8 ov[KS], gv[KS];
  if (D != 256 && dh == D) {
    char* const st = smem + 2 * w * STAGE;
    const int last = nrows - row0 < 32 ? (int)(nrows - row0) - 1 : 31;
    tile_load_async<D == 256 ? 128 : D, 32, 1>(st, a.O + row0 * D, D, 0, last, 0, lane);
    tile_load_async<D == 256 ? 128 : D, 32, 1>(st + STAGE, a.dO + row0 * D, D, 0, last, 0, lane);
    wait_vmem();
    const int z = lq * ROWB + 16 * (hh ^ swz<ROWB>(lq));
#pragma unroll
    for (int ks = 0; ks < KS; ++ks) {
      ov[ks] = lds_b128(st, z ^ (32 * ks));
      gv[ks] = lds_b128(st + STAGE, z ^ (32 * ks));
    }
  } else {
    const long o = (row < nrows ? row : nrows - 1) * dh + 8 * hh;
#pragma unroll
    for (int ks = 0; ks < KS; ++ks)
      if (16 * ks + 8 * hh < dh) {
        ov[ks] = *(const bf16x8*)(a.O + o + 16 * ks);
        gv[ks] = *(const bf16x8*)(a.dO + o + 16 * ks);
      }
  }
  float part = 0.f;
#pragma unroll
  for (int ks = 0; ks < KS; ++ks)
    if (16 * ks + 8 * hh < dh) part = dot8<F16>(ov[ks], gv[ks], part);
  const float d = sum_with_partner32(part);
  if (row < nrows && hh == 0) {
    const long tok = row / a.p.Hq;
    a.Dvec[stat_index(a.p, tok, (int)(row - tok * a.p.Hq))] = d;
  }
}
template <int D, bool F16>
hipError_t launch_prep(const BwdArgs& a, hipStream_t st) {
  const long nrows = (long)a.p.total_tokens * a.p.Hq;
  hipLaunchKernelGGL((bwd_prep_kernel<D, F16>), dim3((unsigned)((nrows + kPrepRows - 1) / kPrepRows)), dim3(256), 0, st, a);
  return hipGetLastError();
}
template hipError_t launch_prep<64, false>(const BwdArgs&, hipStream_t);
template hipError_t launch_prep<64, true>(const BwdArgs&, hipStream_t);
template hipError_t launch_prep<128, false>(const BwdArgs&, hipStream_t);
template hipError_t launch_prep<128, true>(const BwdArgs&, hipStream_t);

template <int D, bool CAUSAL, bool F16, bool DROPOUT = false, bool PAD = false, bool MASK = false,
          int LOCAL = kNoPattern, int DH = D, int NW = 8, bool SHARED = false, bool RAGGED = false>
__global__ __launch_bounds__(64 * NW) __attribute__((amdgpu_waves_per_eu(D == 128 ? NW / 4 : 2, D == 128 ? NW / 4 : 2))) void
    bwd_dkdv_kernel(BwdArgs a) {
  typedef DkdvPlan<D, MASK, LOCAL, NW, SHARED> Plan;
  __shared__ __attribute__((aligned(1024))) char smem[Plan::SMEM];
  dkdv_work<D, CAUSAL, F16, DROPOUT, PAD, MASK, LOCAL, DH, NW, SHARED, RAGGED>(a, smem, {blockIdx.x, Plan::SLOTS});
}
template <int D, bool CAUSAL, bool F16, bool DROPOUT = false, bool PAD = false, bool MASK = false, int LOCAL = kNoPattern,
          bool OWN_D = false, int DH = D, int NW = 8, bool RAGGED = false>
__global__ __launch_bounds__(64 * NW) __attribute__((amdgpu_waves_per_eu(2, 2))) void bwd_dq_kernel(BwdArgs a) {
  typedef DqPlan<D, MASK, LOCAL, NW> Plan;
  __shared__ __attribute__((aligned(1024))) char smem[Plan::SMEM];
  dq_work<D, CAUSAL, F16, DROPOUT, PAD, MASK, LOCAL, OWN_D, DH, NW, RAGGED>(a, smem, {blockIdx.x, Plan::SLOTS});
}

// Whether the four-wavefront form of a backward kernel is taken: workgroups of 128 rows (keys) instead of 256, the
// program of the eight-wavefront form's group 0; at d = 64 two of them fit on a compute unit.
//  * The whole grid of small workgroups fits the 256 compute units at once (MI355X, backward, from the larger to the
//    smaller form in both kernels at d = 64: 1 x 512, 8 heads: 35 -> 30 us; 1 x 4096, 8 heads: 170 -> 153; 2 x 1000,
//    16 heads 55 -> 49; at d = 128 the dK/dV kernel alone: 1 x 1531, 32 heads on 8: 287 -> 262; the dQ kernel
//    does not gain there).
//  * `two` (two fit on a compute unit) and there are many of them: where blocks of 256 would be mostly padding
//    (16 x 300, 32 heads, no mask: 107 -> 86 us), and in the causal dK/dV kernel (`short_too`), whose 128-key blocks
//    also start closer to the diagonal, up to 4096 keys (16k tokens, N = 512: 304 -> 284 us, 2048: 584 -> 572,
//    4096: 980 -> 975, 8192: 1779 -> 1807).
// The plain kernels have the form, and dropout's dK/dV kernel at d = 64. Dropout's dQ kernel, windows, masks, patterns
// and padded head dimensions keep blocks of 256 rows on small grids too: no small form of theirs has been measured, and each
// would be another instantiation per element type and causal flag.
static bool small_workgroups(int n, int pairs, bool short_too, bool two = true) {
  const long small = (long)((n + 127) / 128) * pairs, large = (long)((n + 255) / 256) * pairs;
  if (small <= 256) return true;
  if (!two) return false;
  if (short_too && n <= 4096) return true;
  return large >= 512 && 2 * large * 5 >= 6 * small;
}

// Blocks of `rows` rows (keys) over all pairs of a problem: those that exist, on average in a packed batch.
static double block_count(const Problem& p, int n, long total, int rows, int heads) {
  if (p.cu_seqlens) return ((double)total / rows + 0.5 * p.nseq) * heads;
  return (double)((n + rows - 1) / rows) * heads * p.nseq;
}
static double row_blocks(const BwdArgs& a, int rows) { return block_count(a.p, a.p.N, a.p.total_tokens, rows, a.p.Hq); }
static double key_blocks(const BwdArgs& a, int keys) { return block_count(a.p, a.p.Nk, a.key_rows, keys, a.p.Hkv); }
// An average sequence's length over the longest's.
static double average_part(const Problem& p, int n, long total) { return p.cu_seqlens ? (double)total / ((double)p.nseq * n) : 1; }

// Whether the plain kernels (and dropout's at d = 64) of a joint grid take four wavefronts, blocks of 128 rows and keys.
//  * d = 64, two such workgroups on a compute unit: while the blocks of keys are at most two rounds (MI355X, us of forward and
//    backward in eight wavefronts and four: half precision, dropout, 4 x 1777, 16 heads: 343 and 329; 18 packed of up to 1134,
//    16 heads on 2: 293 and 273; 2 x 325, 2 heads: 25.0 and 23.0; beyond: 4 x 2048, 32 heads: 609 and 621), causal up to 4096 keys as
//    in the two launches.
//  * d = 128, one workgroup on a compute unit either way: a block is a shorter chain (1.06 us a row tile of a block of keys instead of
//    1.2, 1.2 a key block of a block of rows instead of 1.5, about 6 to start), but four wavefronts get through less. The longest
//    chain, or all the work over the compute units and half of a last block, whichever is longer, is within 3% of the better form on
//    44 shapes (1 x 2048, 8 heads: 123 and 115; 3 x 700, 8 heads: 54.5 and 73.0; 2 x 1024, 32 heads on 8: 218 and 198).
bool joint_small(const BwdArgs& a, int D, int causal) {
  const Problem& p = a.p;
  const double keys4 = key_blocks(a, 128);
  if (D == 64) return keys4 <= 1024 || (causal && p.Nk <= 4096);
  const double tiles = (double)((p.N + 31) / 32) * p.G, blocks = (p.Nk + 63) / 64, start = 6;  // of the longest chains
  const double seen = causal ? 0.55 : 1;  // an average block's part of them
  const double part_rows = seen * average_part(p, p.N, p.total_tokens), part_keys = seen * average_part(p, p.Nk, a.key_rows);
  auto estimate = [&](double nk, double nq, double per_tile, double per_block) {
    const double chain = start + tiles * per_tile, row_block = start + blocks * per_block;
    double all = (part_rows * nk * tiles * per_tile + part_keys * nq * blocks * per_block + start * (nk + nq)) / 256;
    if (nk + nq > 256) all += 0.5 * (causal ? 0.2 : 1) * row_block;
    return chain > all ? chain : all;
  };
  return estimate(keys4, row_blocks(a, 128), 1.06, 1.2) < estimate(key_blocks(a, 256), row_blocks(a, 256), 1.2, 1.5);
}

// How long `first` equal blocks of t1 and then `second` of t2 take when `places` workgroups are resident and the next block goes to
// whichever ends first.
static double two_kinds(double first, double t1, double second, double t2, double places) {
  const double full = __builtin_floor(first / places), late = first - full * places;  // late: places that take one more of the first kind
  const double free[2] = {full * t1, late > 0 ? (full + 1) * t1 : full * t1};
  auto done = [&](double t) {  // blocks of the second kind that have ended
    auto of_a_place = [&](double from) { return t < from ? 0. : __builtin_floor((t - from) / t2 + 1e-6); };
    return (places - late) * of_a_place(free[0]) + late * of_a_place(free[1]);
  };
  if (done(free[1]) >= second) return free[1];
  // no earlier than if blocks could be divided, and a whole number of blocks after some place was free
  const double least = (second * t2 + (places - late) * free[0] + late * free[1]) / places;
  double end = free[1] + __builtin_ceil(second / places) * t2;
  for (double from : free)
    for (double i = __builtin_ceil((least - from) / t2 - 1e-6); from + i * t2 < end; ++i)
      if (done(from + i * t2) >= second) end = from + i * t2;
  return end;
}

// Where all blocks of a kind take as long (dense batches without a mask of the causal kind): whether the one grid ends before the two
// launches do. Rests alone do not say so: two kinds of half a round and more make two rounds either way, and blocks of 256 rows of which
// few exist may be the longer part. Blocks take what joint_small says they do (d = 64: 1.5 us a row tile, 1 a key block, 6 to start),
// with dropout 1.6 times as long, and there 5% less in the four wavefronts that only the one grid has for both kinds at d = 64; 2 us lie
// between two launches; the pre-pass takes 3.5 and the part of its bytes that the dQ kernel does not save. Against the better of the
// two forms on 551 random shapes (MI355X, the backward, queries and keys of one length and of two, masks, patterns, dropout) this takes
// 0.3% longer on average, the rests alone 1.3% (us, one grid and two launches: 32 x 44 queries on 3127 keys, 16 heads on 2 of 64: 196 and
// 147; 18 x 103 on 585, 32 on 16 of 64: 84.5 and 74.7; 25 x 268, 32 heads of 64: 158 and 125; 2 x 199 on 8152, 8 heads of 128, mask: 362 and
// 329; where it stays: 10 x 934 on 54, 32 on 16 of 64, mask: 91.5 and 107; half precision, dropout, 4 x 1777, 16 heads of 64: 263 and 274).
static bool joint_sooner(const BwdArgs& a, int D, bool small) {
  const Problem& p = a.p;
  const bool plain = p.d == D && !p.mask && !p.bmask;
  if (D == 128 && plain && !p.drop_thr) small = joint_small(a, D, false);
  const double rows = (double)p.N, keys = (double)p.Nk, slower = p.drop_thr ? 1.6 : 1;
  auto key_time = [&](bool four) {
    return 6 + slower * p.G * (D == 64 ? 1.5 * __builtin_ceil(rows / 64) : (four ? 1.06 : 1.2) * __builtin_ceil(rows / 32));
  };
  auto row_time = [&](bool four) { return 6 + slower * (D == 64 ? 1. : four ? 1.2 : 1.5) * __builtin_ceil(keys / 64); };
  auto places = [&](bool four) { return D == 64 && four ? 512 : 256; };
  const bool shared = D == 128 && p.drop_thr && dropout_shared(p, false);
  auto blocks_of_keys = [&](bool four) { return key_blocks(a, four || p.mask || shared ? 128 : 256); };
  auto blocks_of_rows = [&](bool four) { return row_blocks(a, four ? 128 : 256); };
  const double pre_pass = 3.5 + 0.6 * p.total_tokens * (double)p.Hq * p.d * 4 / 4e6;  // (bytes at 4 TB/s)
  const double one = two_kinds(blocks_of_keys(small), key_time(small), blocks_of_rows(small), row_time(small), places(small)) + pre_pass;
  // (the forms that launch_dq and launch_dkdv take)
  const bool four_q = D == 64 && plain && !p.drop_thr && small_workgroups(p.N, p.Hq * p.nseq, false);
  const bool four_k = plain && (D == 64 || !p.drop_thr) && small_workgroups(p.Nk, p.Hkv * p.nseq, false, D == 64);
  const double two = __builtin_ceil(blocks_of_rows(four_q) / places(four_q)) * row_time(four_q) +
                     __builtin_ceil(blocks_of_keys(four_k) / places(four_k)) * key_time(four_k) + 2;
  return (small && D == 64 && p.drop_thr ? 0.95 : 1) * one < two;
}

// Whether the backward is one grid (fa_bwd_joint.h) or two launches. The one grid costs the pre-pass (a pass over O and dO, 1 to 4% of
// the backward, part of which the dQ kernel saves) and gains what the two launches leave idle: the rest of their last rounds, and
// under the causal mask, whose blocks are uneven, whatever a grid of one round does not fill. MI355X, us of forward and backward, two
// launches and one grid: 2 x 2304, 1 head of 128: 180 -> 124; 1 x 448, 8 heads on 4 of 64: 42.0 -> 33.7; 3 x 2402, 4 heads on 1 of
// 128, window of 95: 103 -> 87; 7 x 1152, 16 heads on 8 of 128: 436 -> 362; 16 x 1024, 16 heads on 4 of 128: 413 -> 361; 27 x 600, 16
// heads of 128: 515 -> 492. Rounds without a rest are better off as they were: 8 x 2048, 32 heads of 64: 732 and 750; 4 x 1024, 16 heads
// of 128, window of 129: 77.8 and 81.0; 32 x 256, 16 heads of 96: 125 and 129. Packed batches, whose blocks nobody has counted: up to
// four rounds of blocks of keys (9 of up to 2077, 16 heads on 8 of 64: 286 -> 266; 16 of up to 4096, 32 heads on 8 of 128: even;
// the backward alone, of two lengths: 16 x 4096 on 128, 16 heads of 64: 214 -> 168; 10 of up to 382 on up to 8030, 4 heads of 128, causal, five
// rounds: 278 in two launches, 356).
bool joint_form(const BwdArgs& a, int D, int causal) {
  const Problem& p = a.p;
  const bool small = D == 64 && p.d == D && !p.mask && !p.bmask && !windowed(p) && joint_small(a, D, causal);
  const int rows = small ? 128 : 256, keys = p.mask ? 128 : rows, slots = small ? 512 : 256;
  const double key_rounds = key_blocks(a, keys) / slots, row_rounds = row_blocks(a, rows) / slots;
  if (p.cu_seqlens) return key_rounds < 4;
  auto rest = [](double rounds) { return __builtin_ceil(rounds) - rounds; };
  const bool idle = (causal && key_rounds <= 1) || rest(key_rounds) + rest(row_rounds) > 0.04 * (key_rounds + row_rounds);
  return idle && (causal || windowed(p) || joint_sooner(a, D, small));
}

// How many workgroups share the row tiles of a block of keys (1: one takes all of them). A block's chain is G * N / 32 tiles (64 at
// d = 64) long, G times that of a block of rows, and few key/value heads make few blocks: the chip waits for a handful of
// workgroups. Shares leave float32 sums that merge_keys_kernel adds: a write and a read of 8 bytes an element and a launch.
// Estimated in us as in joint_small, with eight wavefronts: the longest chain, or all the work over the compute units; taken
// where it saves a fifth. MI355X, us of forward and backward, without and with: 1 x 8192, 8 heads on 1 of 128, causal: 2793 -> 728; 1 x
// 2048, 32 heads on 8 of 128: 391 -> 193, of 64: 231 -> 117; 2 x 817, 8 heads on 1 of 128: 273 -> 62; window of 512, 1 x 6000, 8 heads on 1 of
// 128: 311 -> 114; dropout, 2 x 3000, 8 heads on 1 of 64: 842 -> 258; 8 packed of up to 1500, 32 heads on 4 of 64: 361 -> 233. Where
// nothing is idle it is left: 8 x 1024, 16 heads on 4 of 128.
// Only for groups of four heads and more, with some thousand rows to a block of keys (share_rows): the sums are rounded in another order
// than a single chain's, and with fewer heads or shorter sequences, which gain less, a sequence has the same gradients in every batch
// (what that leaves: 1 x 1024, 4 heads on 1 of 64: 121, with shares 45; 4 x 600 of 128: 127, with shares 53). Not for masks and
// patterns, nor for packed batches of two lengths.
static int key_shares(const BwdArgs& a, int D, int causal) {
  const Problem& p = a.p;
  if (!a.partial || p.mask || p.bmask || p.cu_seqlens_k) return 1;
  const long room = share_rows(a.key_rows, p.Hq, p.Hkv, p.N);
  if (!room) return 1;
  const int most = (int)(room / (a.key_rows * p.Hkv));
  const bool window = windowed(p) && p.win_left >= 0 && p.win_right >= 0;
  const double seen = window ? p.win_left + p.win_right + 256. : 1e9;  // rows that see a block of keys, keys that a block of rows sees
  const double rows = p.N < seen ? p.N : seen, keys = p.Nk < seen ? p.Nk : seen, start = 6;
  const double chain = rows * p.G * (D == 64 ? 1.5 / 64 : 1.2 / 32), row_block = start + keys / 64 * (D == 64 ? 1.0 : 1.5);
  const double nk = key_blocks(a, 256), nq = row_blocks(a, 256);
  const double part = (causal ? 0.55 : 1) * average_part(p, p.N, p.total_tokens);  // an average one
  const double work = part * (nk * chain + nq * row_block) / 256, merged = a.key_rows * p.Hkv * (double)p.d * 8 / 4e6;
  int best = 1;
  double least = (start + chain > work ? start + chain : work) * 0.8;
  for (int z = 2; z <= most; ++z) {
    double t = start + chain / z;
    if (t < row_block) t = row_block;
    const double all = work + start * z * nk / 256 + 0.5 * (nk * z + nq > 256 ? t : 0);
    if (t < all) t = all;
    t += 4 + z * merged;
    if (t < least) {
      least = t;
      best = z;
    }
  }
  return best;
}

// dK, dV from the sums of the shares: eight elements a thread, the scaling with dK. Bound by the bytes of the sums.
template <bool F16>
__global__ __launch_bounds__(256) void merge_keys_kernel(BwdArgs a) {
  const long n = a.key_rows * a.p.Hkv * a.p.d, i = 8 * ((long)blockIdx.x * 256 + threadIdx.x);
  if (i >= n) return;
  const bool v = blockIdx.y != 0;
  const float* src = a.partial + (v ? n : 0) + i;
  f32x4 lo = {0, 0, 0, 0}, hi = {0, 0, 0, 0};
#pragma unroll 4
  for (int z = 0; z < a.shares; ++z) {
    lo += *(const f32x4*)(src + 2 * n * z);
    hi += *(const f32x4*)(src + 2 * n * z + 4);
  }
  const float mul = v ? 1.f : a.p.scale;
  u32x4 o;
  o[0] = pack2<F16>(lo[0] * mul, lo[1] * mul);
  o[1] = pack2<F16>(lo[2] * mul, lo[3] * mul);
  o[2] = pack2<F16>(hi[0] * mul, hi[1] * mul);
  o[3] = pack2<F16>(hi[2] * mul, hi[3] * mul);
  *(u32x4*)((v ? a.dV : a.dK) + i) = o;
}
hipError_t launch_merge_keys(const BwdArgs& a, hipStream_t st) {
  const long n = a.key_rows * a.p.Hkv * a.p.d;
  const dim3 grid((unsigned)((n / 8 + 255) / 256), 2), block(256);
  if (a.p.f16) hipLaunchKernelGGL((merge_keys_kernel<true>), grid, block, 0, st, a);
  else hipLaunchKernelGGL((merge_keys_kernel<false>), grid, block, 0, st, a);
  return hipGetLastError();
}

// The dQ kernel. OWN_D: it sums D on the way (the whole backward, with every option); otherwise the pre-pass has (the
// separate stages, which have no options). RAGGED: a.p.cu_seqlens is set (the stages and the two patterns of the mask
// are for dense batches).
template <int D, bool F16, bool OWN_D, bool RAGGED>
static hipError_t launch_dq(const BwdArgs& a, int causal, hipStream_t st) {
  constexpr int DN = dn_of(D);
  const int pairs = a.p.Hq * a.p.nseq;
  const dim3 grid(grid_size(a.p, (a.p.N + 255) / 256, a.p.Hq, kXcdUnits)), block(512);
  if constexpr (OWN_D && !RAGGED) {
    if (a.p.bmask) {  // block-sparse pattern (perhaps with a window)
      hipLaunchKernelGGL((bwd_dq_kernel<D, false, F16, false, false, false, kBlocks, true>), grid, block, 0, st, a);
      return hipGetLastError();
    }
    if (a.p.mask) {
      if (causal) hipLaunchKernelGGL((bwd_dq_kernel<D, true, F16, false, false, true, kNoPattern, true>), grid, block, 0, st, a);
      else hipLaunchKernelGGL((bwd_dq_kernel<D, false, F16, false, false, true, kNoPattern, true>), grid, block, 0, st, a);
      return hipGetLastError();
    }
  }
  if constexpr (OWN_D) {
    if (windowed(a.p)) {
      hipLaunchKernelGGL((bwd_dq_kernel<D, false, F16, false, false, false, kWindow, true, D, 8, RAGGED>), grid, block, 0, st, a);
      return hipGetLastError();
    }
    if (a.p.drop_thr) {  // (the entry points keep dropout away from padded head dimensions)
      if (causal) hipLaunchKernelGGL((bwd_dq_kernel<D, true, F16, true, false, false, kNoPattern, true, D, 8, RAGGED>), grid, block, 0, st, a);
      else hipLaunchKernelGGL((bwd_dq_kernel<D, false, F16, true, false, false, kNoPattern, true, D, 8, RAGGED>), grid, block, 0, st, a);
      return hipGetLastError();
    }
  }
  if (a.p.d != D && a.p.d <= DN) {
    if (causal) hipLaunchKernelGGL((bwd_dq_kernel<D, true, F16, false, true, false, kNoPattern, OWN_D, DN, 8, RAGGED>), grid, block, 0, st, a);
    else hipLaunchKernelGGL((bwd_dq_kernel<D, false, F16, false, true, false, kNoPattern, OWN_D, DN, 8, RAGGED>), grid, block, 0, st, a);
    return hipGetLastError();
  }
  if (a.p.d != D) {
    if (causal) hipLaunchKernelGGL((bwd_dq_kernel<D, true, F16, false, true, false, kNoPattern, OWN_D, D, 8, RAGGED>), grid, block, 0, st, a);
    else hipLaunchKernelGGL((bwd_dq_kernel<D, false, F16, false, true, false, kNoPattern, OWN_D, D, 8, RAGGED>), grid, block, 0, st, a);
    return hipGetLastError();
  }
  if constexpr (D == 64) {
    if (small_workgroups(a.p.N, pairs, false)) {
      const dim3 sgrid(grid_size(a.p, (a.p.N + 127) / 128, a.p.Hq, 2 * kXcdUnits));
      if (causal) hipLaunchKernelGGL((bwd_dq_kernel<D, true, F16, false, false, false, kNoPattern, OWN_D, D, 4, RAGGED>), sgrid, dim3(256), 0, st, a);
      else hipLaunchKernelGGL((bwd_dq_kernel<D, false, F16, false, false, false, kNoPattern, OWN_D, D, 4, RAGGED>), sgrid, dim3(256), 0, st, a);
      return hipGetLastError();
    }
  }
  if (causal) hipLaunchKernelGGL((bwd_dq_kernel<D, true, F16, false, false, false, kNoPattern, OWN_D, D, 8, RAGGED>), grid, block, 0, st, a);
  else hipLaunchKernelGGL((bwd_dq_kernel<D, false, F16, false, false, false, kNoPattern, OWN_D, D, 8, RAGGED>), grid, block, 0, st, a);
  return hipGetLastError();
}

// The dK/dV kernel.
template <int D, bool F16, bool RAGGED>
static hipError_t launch_dkdv(const BwdArgs& a, int causal, hipStream_t st) {
  constexpr int DN = dn_of(D);
  const int pairs = a.p.Hkv * a.p.nseq;
  const int bck = dkdv_block_keys(a.p.mask != nullptr);  // keys per workgroup differ between the instantiations
  const dim3 grid(grid_size(a.p, (a.p.Nk + bck - 1) / bck, a.p.Hkv, kXcdUnits)), block(512);
  const dim3 sgrid(grid_size(a.p, (a.p.Nk + 127) / 128, a.p.Hkv, (D == 64 ? 2 : 1) * kXcdUnits));
  if constexpr (!RAGGED) {
    if (a.p.bmask) {  // block-sparse pattern (perhaps with a window)
      hipLaunchKernelGGL((bwd_dkdv_kernel<D, false, F16, false, false, false, kBlocks>), grid, block, 0, st, a);
      return hipGetLastError();
    }
    if (a.p.mask) {
      if (causal) hipLaunchKernelGGL((bwd_dkdv_kernel<D, true, F16, false, false, true>), grid, block, 0, st, a);
      else hipLaunchKernelGGL((bwd_dkdv_kernel<D, false, F16, false, false, true>), grid, block, 0, st, a);
      return hipGetLastError();
    }
  }
  if (windowed(a.p)) {
    hipLaunchKernelGGL((bwd_dkdv_kernel<D, false, F16, false, false, false, kWindow, D, 8, false, RAGGED>), grid, block, 0, st, a);
    return hipGetLastError();
  }
  if (a.p.d != D && a.p.d <= DN) {
    if (causal) hipLaunchKernelGGL((bwd_dkdv_kernel<D, true, F16, false, true, false, kNoPattern, DN, 8, false, RAGGED>), grid, block, 0, st, a);
    else hipLaunchKernelGGL((bwd_dkdv_kernel<D, false, F16, false, true, false, kNoPattern, DN, 8, false, RAGGED>), grid, block, 0, st, a);
    return hipGetLastError();
  }
  if (a.p.d != D) {
    if (causal) hipLaunchKernelGGL((bwd_dkdv_kernel<D, true, F16, false, true, false, kNoPattern, D, 8, false, RAGGED>), grid, block, 0, st, a);
    else hipLaunchKernelGGL((bwd_dkdv_kernel<D, false, F16, false, true, false, kNoPattern, D, 8, false, RAGGED>), grid, block, 0, st, a);
    return hipGetLastError();
  }
  const bool small = small_workgroups(a.p.Nk, pairs, D == 64 && causal, D == 64);
  if (a.p.drop_thr) {
    // Dropout at d = 64 takes the four-wavefront form by the same rule (bfloat16, 14 x 353
    // causal, 8 heads on 4, forward + backward: 66.6 us in blocks of 256 keys, 61.5 so).
    if constexpr (D == 128) {
      // (causal or packed, grids as small as that are joint ones: joint_form)
      if constexpr (!RAGGED)
        if (!causal && dropout_shared(a.p, causal)) {
          hipLaunchKernelGGL((bwd_dkdv_kernel<D, false, F16, true, false, false, kNoPattern, D, 8, true, false>), sgrid, block, 0, st, a);
          return hipGetLastError();
        }
    } else if (small) {
      if (causal) hipLaunchKernelGGL((bwd_dkdv_kernel<D, true, F16, true, false, false, kNoPattern, D, 4, false, RAGGED>), sgrid, dim3(256), 0, st, a);
      else hipLaunchKernelGGL((bwd_dkdv_kernel<D, false, F16, true, false, false, kNoPattern, D, 4, false, RAGGED>), sgrid, dim3(256), 0, st, a);
      return hipGetLastError();
    }
    if (causal) hipLaunchKernelGGL((bwd_dkdv_kernel<D, true, F16, true, false, false, kNoPattern, D, 8, false, RAGGED>), grid, block, 0, st, a);
    else hipLaunchKernelGGL((bwd_dkdv_kernel<D, false, F16, true, false, false, kNoPattern, D, 8, false, RAGGED>), grid, block, 0, st, a);
    return hipGetLastError();
  }
  if constexpr (D == 64 || !RAGGED)  // (at d = 128, packed or causal, a grid as small as that is a joint one; single stages are for bfloat16)
    if (small) {
      if (!causal) {
        hipLaunchKernelGGL((bwd_dkdv_kernel<D, false, F16, false, false, false, kNoPattern, D, 4, false, RAGGED>), sgrid, dim3(256), 0, st, a);
        return hipGetLastError();
      }
      if constexpr (D == 64 || !F16) {
        hipLaunchKernelGGL((bwd_dkdv_kernel<D, true, F16, false, false, false, kNoPattern, D, 4, false, RAGGED>), sgrid, dim3(256), 0, st, a);
        return hipGetLastError();
      }
    }
  if (causal) hipLaunchKernelGGL((bwd_dkdv_kernel<D, true, F16, false, false, false, kNoPattern, D, 8, false, RAGGED>), grid, block, 0, st, a);
  else hipLaunchKernelGGL((bwd_dkdv_kernel<D, false, F16, false, false, false, kNoPattern, D, 8, false, RAGGED>), grid, block, 0, st, a);
  return hipGetLastError();
}

// The dQ kernel reads Q, K, V, O that the forward pass has just streamed through the last-level cache (256 MB):
// it goes through the pairs from the last to the first and finds the newest there first (16k tokens, 32 heads of 64,
// MI355X, backward: N = 256 250 -> 235 us, N = 512 without the mask 337 -> 326 us, N >= 1024 -1% .. 0).
template <int D, bool F16>
static hipError_t launch_bwd_d(const BwdArgs& a, int causal, int stages, hipStream_t st) {
  // The whole backward: one launch (short sequences), shares, one grid behind the pre-pass, or two launches, of which the dQ
  // kernel goes first and computes D on the way and the dK/dV kernel reads it.
  // Short sequences at d = 64 are one launch, which keeps D to itself (its store costs 1% of a short step: 14.4 -> 14.5 us for the
  // forward and backward of 1 x 128, 2 heads): not for a caller that may read D afterwards.
  if constexpr (D == 64)
    if (stages == 7 && !a.keep_d && a.p.d == D && !a.p.mask && !a.p.bmask && !windowed(a.p) && !a.p.drop_thr &&
        bwd_short_form(a.p, causal))
      return launch_bwd_short(a, causal, st);
  if (stages == 7) {
    BwdArgs shared = a;
    shared.shares = key_shares(a, D, causal);
    shared.share_turn = a.p.cu_seqlens ? 3 : (int)((a.p.Nk + 255L) / 256 * a.p.Hkv * a.p.nseq % kXcds);  // (packed: nobody has counted the blocks)
    if (shared.shares > 1) return launch_joint_shares<D, F16>(shared, causal, st);
  }
  if (stages == 7 && joint_form(a, D, causal)) return launch_joint<D, F16>(a, causal, st);
  if (stages == 7 && a.p.cu_seqlens) {
    if (hipError_t e = launch_dq<D, F16, true, true>(a, causal, st)) return e;
    return launch_dkdv<D, F16, true>(a, causal, st);
  }
  if (stages == 7) {
    if (hipError_t e = launch_dq<D, F16, true, false>(a, causal, st)) return e;
    return launch_dkdv<D, F16, false>(a, causal, st);
  }
  if constexpr (F16) {
    return hipErrorInvalidValue;
  } else {  // one stage or two (fa_bwd_stages: dense batches in bfloat16)
    if (stages & 1)
      if (hipError_t e = launch_prep<D, F16>(a, st)) return e;
    if (stages & 2)
      if (hipError_t e = launch_dkdv<D, F16, false>(a, causal, st)) return e;
    if (stages & 4)
      if (hipError_t e = launch_dq<D, F16, false, false>(a, causal, st)) return e;
    return hipSuccess;
  }
}

hipError_t launch_bwd(const BwdArgs& a, int d, int causal, int stages, hipStream_t st) {
  if (stages & 4)
    if (hipError_t e = launch_keyless_rows(a.p, a.dQ, nullptr, st)) return e;
  if (d == 256) {  // (the two kernels live in fa_d256.hip)
    if (stages != 7 && (stages & 1))  // the D pre-pass is the generic one
      if (hipError_t e = launch_prep<256, false>(a, st)) return e;
    return launch_bwd256(a, causal, stages, st);
  }
  if (a.p.f16) return d <= 64 ? launch_bwd_d<64, true>(a, causal, stages, st) : launch_bwd_d<128, true>(a, causal, stages, st);
  return d <= 64 ? launch_bwd_d<64, false>(a, causal, stages, st) : launch_bwd_d<128, false>(a, causal, stages, st);
}

}  // namespace fa
