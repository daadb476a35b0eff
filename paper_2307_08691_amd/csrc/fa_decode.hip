// Forward for very few query rows against many keys (decoding: one or a few new tokens per
// sequence against a key/value cache; the inference setting of the multi-query / grouped-query
// paragraph of section 3.1). Algorithm 1 with the parallelism turned round: the rows of one
// (sequence, key/value head) — query row x query head of the group, at most 32 — fit ONE 32-row
// MFMA tile, so there is nothing to split over wavefronts along the rows. Instead the eight (or four)
// wavefronts of a workgroup take the KEY tiles (32 keys each) of the workgroup's share of the keys
// in turn, every wavefront with a running softmax of its own (m, l, O), without a barrier inside
// the loop; at the end the partial results are combined through LDS with the identity the
// paper uses between blocks (section 3.1.1) and the workgroup writes its share's normalised
// partial O and logsumexp, which fwd_merge_kernel combines over the shares as for the split kernel.
// The pass is bound by HBM: K and V are read once, and the point of the layout is to keep eight
// independent streams of loads in flight per compute unit.
//
// Per 32-key tile and wavefront: K_j goes straight from memory into the A-operand registers of
// S^T = K_j Q^T (lane (key, half) fetches 16 bytes of its key's row per contraction step), V_j goes
// memory -> LDS by direct copies into a tile private to the wavefront and is read back transposed
// as the A operand of O^T += V_j^T P^T. Both are requested one tile ahead (two register sets,
// two LDS tiles per wavefront). The K loads are ordinary loads (the compiler waits for them where
// they are used); the V copies are the hand-issued direct-to-LDS copies of fa_lds.h, which the
// compiler does not see: one s_waitcnt vmcnt(0) per tile, after the tile's work, covers them.
//
// Small batches are a chain of memory latencies: lengths, page table, Q, tiles, then the merge. So all lengths come with one load,
// a wavefront's pages with one, its first two tiles are requested together, and the merge requests four shares at a time
// (MI355X, 4 sequences of up to 2048 keys, 32 heads on 8, d = 128, both kernels replayed from a graph: 16.3 -> 14.0 us with
// all four; 64 paged sequences of up to 8192: 236 -> 233), and up to sixteen shares in the merge, logsumexps and partial rows
// together, since (2 sequences of up to 7168, 16 heads on 8 of 64: 12.5 -> 11.2; 3 of up to 14592, 4 heads on 1 of 64: 14.6 -> 13.3).
#include <hip/hip_runtime.h>

#include <type_traits>

#include "fa_kernels.h"
#include "fa_lds.h"

namespace fa {

// TWO: two workgroups fit on a compute unit, so that one's start (lengths, pages, first tiles: a chain of memory latencies) and end
// pass while the other streams. At d = 64 the eight wavefronts then have 128 registers each, at d = 128, where the V tiles of eight fill
// the LDS, a workgroup has four. Taken by decode_two below.
constexpr int decode_waves(int D, bool two) { return two && D == 128 ? 4 : 8; }
template <int D, bool CAUSAL, bool F16, bool TWO>
__global__ __launch_bounds__(64 * decode_waves(D, TWO)) __attribute__((amdgpu_waves_per_eu(TWO && D == 64 ? 4 : 2, TWO && D == 64 ? 4 : 2))) void
    fwd_decode_kernel(FwdArgs a) {
  constexpr int NW = decode_waves(D, TWO);
  constexpr bool TIGHT = TWO && D == 64;  // (128 registers)
  constexpr int KT = 32;             // keys per tile
  constexpr int KS = D / 16;         // contraction steps of the first product
  constexpr int DT = D / 32;         // 32-row tiles of O^T
  constexpr int ROWB = 2 * D;
  constexpr int TILEB = KT * ROWB;   // one V tile
  constexpr int WAVEB = 2 * TILEB;   // a wavefront's two V tiles; later its partial O^T (D x 32 floats)
  static_assert(WAVEB == D * 32 * 4, "the partial O^T of a wavefront takes the place of its two V tiles");
  constexpr int STAT_OFF = NW * WAVEB;  // m and l of the wavefronts: [2][NW][32] floats
  __shared__ __attribute__((aligned(1024))) char smem[STAT_OFF + 2 * NW * 32 * 4];

  const Problem& p = a.p;
  const int tid = threadIdx.x, lane = tid & 63;
  const int w = __builtin_amdgcn_readfirstlane(tid >> 6);
  const int lq = lane & 31, hh = lane >> 5;
  const int nsplit = a.nsplit;
  // All shares of a pair on one XCD, an XCD's pairs one after the other. (No two workgroups read the same keys, but with a pair's
  // shares on all XCDs small batches are slower: 1 sequence of up to 2816 keys, 2 heads on 1: 13.6 us so, 14.6 spread; 3 of up to 7168,
  // 32 heads on 8 of 64: 12.9 and 13.5.)
  const int k = blockIdx.x / kXcds, turn = k / nsplit;
  const int pair = turn * kXcds + blockIdx.x % kXcds, rank = pair / p.Hkv;
  const int split = k - turn * nsplit, g = pair - rank * p.Hkv;
  if (rank >= p.nseq) return;
  // (sequences of uneven cache lengths are handed out longest first)
  const CacheSequence cs = cache_sequence(a, rank);
  const int s = cs.s;
  const SeqInfo si = seq_info(p, s);
  const int n = si.n, nk = cs.len;
  // With a single share there is nothing to merge: the workgroup writes O and LSE themselves (and
  // the launch leaves fwd_merge_kernel out), also for a sequence without keys.
  const bool direct = nsplit == 1;
  if (n == 0) return;
  if (nk == 0) {  // (several shares: L = -inf tells fwd_merge_kernel, which fills the rows)
    if (!direct) {
      if (tid < n * p.G)
        a.Lpart[(long)split * p.total_tokens * p.Hq + s * p.lse_seq_stride + (long)(g * p.G + tid % p.G) * p.lse_head_stride + tid / p.G] = -INFINITY;
    } else {
      for (int i = tid; i < n * p.G * (D / 8); i += 64 * NW) {  // 16-byte pieces of the rows of this key/value head
        const int prow_ = i / (D / 8), q_ = prow_ / p.G, h_ = g * p.G + prow_ % p.G;
        *(u32x4*)(a.O + ((si.tok0 + q_) * p.Hq + h_) * D + 8 * (i % (D / 8))) = (u32x4){0, 0, 0, 0};
        if (i % (D / 8) == 0) a.LSE[s * p.lse_seq_stride + (long)h_ * p.lse_head_stride + q_] = -INFINITY;
      }
    }
    return;
  }
  const int off = nk - n;
  const int nrows = n * p.G;  // packed rows: query * G + head of the group; at most 32 (the launch checks)

  // this lane's packed row, its query and its head
  const bool row_ok = lq < nrows;
  const int prow = row_ok ? lq : nrows - 1;  // lanes past the end compute on a copy and store nothing
  const int row = prow / p.G, h = g * p.G + prow % p.G;
  bf16x8 Qf[KS];
  {
    const __bf16* qp = a.Q + ((si.tok0 + row) * p.Hq + h) * D + 8 * hh;
#pragma unroll
    for (int ks = 0; ks < KS; ++ks) Qf[ks] = *(const bf16x8*)(qp + 16 * ks);
  }

  // the share's keys, in blocks of 64 as in the split kernel (the two kernels split alike), then in tiles of 32
  const int ncol_all = (nk + 63) / 64;
  const int per_split = (ncol_all + nsplit - 1) / nsplit;
  const int jb = split * per_split;
  const int ncol = jb + per_split < ncol_all ? jb + per_split : ncol_all;  // (the last query stands at the last key: no causal bound)
  const long lpart = (long)split * p.total_tokens * p.Hq + s * p.lse_seq_stride + (long)h * p.lse_head_stride + row;
  if (jb >= ncol) {  // no key of this share is visible: L = -inf says so to the merge
    if (w == 0 && row_ok && hh == 0) a.Lpart[lpart] = -INFINITY;
    return;
  }
  const int t_begin = 2 * jb, t_end = (nk + KT - 1) / KT < 2 * ncol ? (nk + KT - 1) / KT : 2 * ncol;  // tiles of 32 keys

  // ---- loads of one tile: K rows into registers, V rows into the wavefront's LDS tile `buf`
  const long kstride = (long)p.Hkv * D;
  char* vbuf = smem + w * WAVEB;
  u32x4 Kr[2][KS];
  const int pmask = a.block_table ? (1 << a.page_log2) - 1 : 0;
  // Pages of this wavefront's tiles t_begin + w + 8 i: lane i % 64 holds the one of tile i. (Looked up one by one each was a
  // memory latency in front of its tile's requests: 50 sequences of up to 7680 keys, 32 heads on 8 of 64: 123 us so, 104 now.)
  // The first two, which the start waits for, go the shorter way of a scalar load. That is even on average: without it 30 paged
  // batches of 1 .. 96 sequences took 0.96 to 1.04 of the time (44 of up to 768 keys, 16 heads of 64: 23.4 us so, 24.2 without;
  // 4 of up to 2048, 32 heads on 8 of 128: 14.1 and 13.7).
  int pages = 0;
  auto load_pages = [&](int t0) {
    const int t = t0 + NW * lane < t_end ? t0 + NW * lane : t_end - 1;
    pages = a.block_table[(long)s * a.table_stride + (t * KT >> a.page_log2)];
  };
  if (a.block_table && t_begin + w + 2 * NW < t_end) load_pages(t_begin + w);
  auto tile_base = [&](int t, const __bf16* pool, int& first, int& last) {  // rows of tile t: base pointer, first row, last valid row
    const int key0 = t * KT;
    if (a.block_table) {
      const int in_page = key0 & pmask;
      const int i = (t - t_begin) / NW;
      const int pg = i < 2 ? __builtin_amdgcn_readfirstlane(a.block_table[(long)s * a.table_stride + (key0 >> a.page_log2)])
                           : __builtin_amdgcn_readlane(pages, i & 63);
      first = in_page;
      last = nk - 1 - (key0 - in_page);
      last = last < pmask ? last : pmask;
      return pool + (((long)pg << a.page_log2) * p.Hkv + g) * D;
    }
    first = key0;
    last = nk - 1;
    return pool + (si.tok0k * p.Hkv + g) * D;
  };
  auto issue = [&](int t, auto BUF) {
    constexpr int buf = decltype(BUF)::value;
    int first, last;
    if (a.block_table && ((t - t_begin) / NW) % 64 == 0 && t >= t_begin + NW) load_pages(t);
    const __bf16* kb = tile_base(t, a.K, first, last);
    int ln = lane;  // (hidden from the compiler, which would keep one address per step)
    if (TIGHT) asm volatile("" : "+v"(ln));
    const int kr = first + (ln & 31) < last ? first + (ln & 31) : last;  // keys past the end repeat the last one (masked below)
    const __bf16* kp = kb + (long)kr * kstride + 8 * (ln >> 5);
#pragma unroll
    for (int ks = 0; ks < KS; ++ks) Kr[buf][ks] = *(const u32x4*)(kp + 16 * ks);
    const __bf16* vb = tile_base(t, a.V, first, last);
    tile_load_async<D, KT, 1>(vbuf + buf * TILEB, vb, kstride, first, last, 0, lane);
  };

  // ---- on-chip state of this wavefront (Algorithm 1, line 5)
  f32x16 O[DT];
#pragma unroll
  for (int dt = 0; dt < DT; ++dt) O[dt] = (f32x16){0};
  float m = -INFINITY, l = 0.f;
  const float c2 = p.scale_log2e;
  const int pos = row + off;  // this lane's query among the keys

  // lane constants of the transposing V reads (see fa_lds.h)
  const int p16 = lane & 15, g16 = (lane >> 4) & 1;
  int zcol[2];
#pragma unroll
  for (int u = 0; u < 2; ++u)
    zcol[u] = swz_off<ROWB>(4 * hh + (p16 >> 2) + 8 * u, 2 * g16 + ((p16 & 3) >> 1)) + 8 * (p16 & 1);

  auto compute = [&](int t, auto BUF) {
    constexpr int buf = decltype(BUF)::value;
    // ---- S^T = K_j Q^T (Algorithm 1, line 8)
    f32x16 S = (f32x16){0};
#pragma unroll
    for (int ks = 0; ks < KS; ++ks) S = mfma32<F16>(__builtin_bit_cast(bf16x8, Kr[buf][ks]), Qf[ks], S);
    // ---- keys past the end and (causal) above the query's position
    const int key0 = t * KT;
    const int lim = (CAUSAL && pos < nk - 1 ? pos : nk - 1) - key0 - 4 * hh;  // last visible key, relative to this lane's first
    if (key0 + KT - 1 > (CAUSAL ? off : nk - 1) || key0 + KT > nk) {
#pragma unroll
      for (int r = 0; r < 16; ++r) S[r] = acc_row(r, 0) > lim ? -INFINITY : S[r];
    }
    // ---- online softmax (Algorithm 1, line 9); a row may have seen no key yet
    float mx = S[0];
#pragma unroll
    for (int r = 1; r < 16; ++r) mx = fmaxf(mx, S[r]);
    mx = max_with_partner32(mx);
    const float m_new = fmaxf(m, mx);
    const float alpha = m_new == -INFINITY ? 1.f : fast_exp2((m - m_new) * c2);
    const float ref = m_new == -INFINITY ? 0.f : m_new * c2;
    float rs = 0.f;
#pragma unroll
    for (int r = 0; r < 16; ++r) {
      S[r] = fast_exp2(__builtin_fmaf(S[r], c2, -ref));
      rs += S[r];
    }
    l = l * alpha + rs;
    m = m_new;
#pragma unroll
    for (int dt = 0; dt < DT; ++dt)
#pragma unroll
      for (int r = 0; r < 16; ++r) O[dt][r] *= alpha;
    bf16x8 Pf[2];
    Pf[0] = pack8<F16>(S, 0);
    Pf[1] = pack8<F16>(S, 1);
    // ---- O^T += V_j^T P^T (Algorithm 1, line 10)
    const int vb = w * WAVEB + buf * TILEB;
#pragma unroll
    for (int i = 0; i < 2 * DT; ++i) {
      const int dt = i >> 1, ro = (16 * (i & 1)) * ROWB;
      const bf16x8 x = lds_tr_pair(smem, ((zcol[0] + vb) ^ (64 * dt)) + ro, ((zcol[1] + vb) ^ (64 * dt)) + ro);
      O[dt] = mfma32<F16>(x, Pf[i & 1], O[dt]);
      if constexpr (TIGHT) __builtin_amdgcn_sched_barrier(0);  // (operands one by one)
    }
  };

  // ---- this wavefront's tiles: t_begin + w, + 8, ...; the next one is requested before the current one is used
  using B0 = std::integral_constant<int, 0>;
  using B1 = std::integral_constant<int, 1>;
  int t = t_begin + w;
  if (t < t_end) {
    // (the first two tiles are requested together: short shares hold no more, and wait once instead of twice)
    issue(t, B0{});
    if (t + NW < t_end) issue(t + NW, B1{});
#pragma unroll
    for (int ks = 0; ks < KS; ++ks) touch(Qf[ks]);
    wait_vmem();
    bool more = t + NW < t_end;  // the next tile is here already
    while (true) {
      if (!more && t + NW < t_end) issue(t + NW, B1{});
      more = false;
      compute(t, B0{});
      asm volatile("s_waitcnt lgkmcnt(0)" ::: "memory");  // the reads of this tile are done before its buffer is requested again
      wait_vmem();
      t += NW;
      if (t >= t_end) break;
      if (t + NW < t_end) issue(t + NW, B0{});
      compute(t, B1{});
      asm volatile("s_waitcnt lgkmcnt(0)" ::: "memory");
      wait_vmem();
      t += NW;
      if (t >= t_end) break;
    }
  }

  // ---- combine the wavefronts (section 3.1.1's rescaling, once more) and write the share's partial result
  const float lsum = sum_with_partner32(l);
  __syncthreads();  // every wavefront is done with its V tiles
  float* part = (float*)(smem + w * WAVEB);  // [d][row]
#pragma unroll
  for (int dt = 0; dt < DT; ++dt)
#pragma unroll
    for (int r = 0; r < 16; ++r) part[(32 * dt + acc_row(r, hh)) * 32 + lq] = O[dt][r];
  float* stat = (float*)(smem + STAT_OFF);
  if (hh == 0) {
    stat[w * 32 + lq] = m;
    stat[32 * NW + w * 32 + lq] = lsum;
  }
  __syncthreads();
  {
    constexpr int CPT = D / (2 * NW);
    int th = tid;  // (recomputed here: nothing of these addresses is to live across the main loop)
    if (TIGHT) asm volatile("" : "+v"(th));
    const int r = th & 31, dg = th >> 5;  // this thread: row r, CPT columns from dg * CPT
    float mm = -INFINITY;
#pragma unroll
    for (int ww = 0; ww < NW; ++ww) mm = fmaxf(mm, stat[ww * 32 + r]);
    float wgt[NW], den = 0.f;
#pragma unroll
    for (int ww = 0; ww < NW; ++ww) {
      const float mw = stat[ww * 32 + r];
      wgt[ww] = mw == -INFINITY ? 0.f : fast_exp2((mw - mm) * c2);
      den += wgt[ww] * stat[32 * NW + ww * 32 + r];
    }
    const bool ok = r < nrows;
    const int prow2 = ok ? r : nrows - 1;
    const int row2 = prow2 / p.G, h2 = g * p.G + prow2 % p.G;
    const float inv = den > 0.f ? 1.f / den : 0.f;  // no visible key in this share: O = 0, L = -inf
    float out[CPT];
#pragma unroll
    for (int i = 0; i < CPT; ++i) {
      const int dcol = dg * CPT + i;
      float acc = 0.f;
#pragma unroll
      for (int ww = 0; ww < NW; ++ww) acc += wgt[ww] * ((const float*)(smem + ww * WAVEB))[dcol * 32 + r];
      out[i] = acc * inv;
    }
    const float lse = den > 0.f ? mm * p.scale + fast_log2(den) * kLn2 : -INFINITY;
    const long lidx = s * p.lse_seq_stride + (long)h2 * p.lse_head_stride + row2;
    if (direct) {  // the final result, rounded to the element type
      if (ok) {
        __bf16* op = a.O + ((si.tok0 + row2) * p.Hq + h2) * D + dg * CPT;
        if constexpr (CPT % 8 == 0) {  // 16 bytes at a time
#pragma unroll
          for (int o8 = 0; o8 < CPT; o8 += 8) {
            u32x4 v;
#pragma unroll
            for (int u = 0; u < 4; ++u) v[u] = pack2<F16>(out[o8 + 2 * u], out[o8 + 2 * u + 1]);
            *(u32x4*)(op + o8) = v;
          }
        } else {  // four columns: 8 bytes
          u32x2 v;
          v[0] = pack2<F16>(out[0], out[1]);
          v[1] = pack2<F16>(out[2], out[3]);
          *(u32x2*)op = v;
        }
        if (dg == 0) a.LSE[lidx] = lse;
      }
    } else if (ok) {
      float* op = a.Opart + (((long)split * p.total_tokens + si.tok0 + row2) * p.Hq + h2) * D + dg * CPT;
#pragma unroll
      for (int i = 0; i < CPT; ++i) op[i] = out[i];
      if (dg == 0) a.Lpart[(long)split * p.total_tokens * p.Hq + lidx] = lse;
    }
  }
}

// `a.nsplit` shares per (sequence, key/value head); N * G <= 32 rows. The caller runs fwd_merge_kernel afterwards.
template <int D, bool TWO>
static hipError_t launch_decode_as(const FwdArgs& a, int causal, unsigned workgroups, hipStream_t st) {
  const dim3 grid(workgroups), block(64 * decode_waves(D, TWO));
  if (a.p.f16) {
    if (causal) hipLaunchKernelGGL((fwd_decode_kernel<D, true, true, TWO>), grid, block, 0, st, a);
    else hipLaunchKernelGGL((fwd_decode_kernel<D, false, true, TWO>), grid, block, 0, st, a);
  } else {
    if (causal) hipLaunchKernelGGL((fwd_decode_kernel<D, true, false, TWO>), grid, block, 0, st, a);
    else hipLaunchKernelGGL((fwd_decode_kernel<D, false, false, TWO>), grid, block, 0, st, a);
  }
  return hipGetLastError();
}
// Whether two workgroups share a compute unit: more workgroups than compute units, and the more of them the longer a share may be,
// up to 2048 keys. (MI355X, us, one and two on a compute unit; uneven lengths, pages of 256, cap keys at most. d = 128: 96 sequences, 32
// heads, 256 keys: 107.6 and 64.3; 64 x 16 heads, 512: 42.2 and 30.3; 64, 32 heads on 8, 768: 25.3 and 21.4; 40 x 16, 1024: 40.1 and 33.1;
// 96 x 32, 2048: 342 and 300; but 40 x 8, 768: 17.1 and 18.5; 24 x 16, 1536: 28.7 and 32.7; 64, 32 on 8, 8192: 209 and 242: there a longest
// share, which streams at half the rate, is what the others wait for. d = 64: 96 x 32, 256: 79.5 and 52.3; 24 x 32, 2048: 48.3
// and 45.0; 96 x 32, 2048: 222 and 180; 40 x 8, 2048: 20.4 and 22.7; 24 x 16, 8192: 107 and 134.)
static bool decode_two(const FwdArgs& a, long workgroups) {
  const int keys = a.p.Nk / a.nsplit;
  return workgroups > 256 && keys <= 2048 && 2 * workgroups >= keys;
}
template <int D>
static hipError_t launch_decode_d(const FwdArgs& a, int causal, hipStream_t st) {
  const int pairs = a.p.Hkv * a.p.nseq;
  const unsigned workgroups = (unsigned)((pairs + kXcds - 1) / kXcds * kXcds * a.nsplit);
  if (decode_two(a, (long)pairs * a.nsplit)) return launch_decode_as<D, true>(a, causal, workgroups, st);
  return launch_decode_as<D, false>(a, causal, workgroups, st);
}

hipError_t launch_fwd_decode(const FwdArgs& a, int d, int causal, hipStream_t st) {
  if (d == 64) return launch_decode_d<64>(a, causal, st);
  if (d == 128) return launch_decode_d<128>(a, causal, st);
  return hipErrorInvalidValue;
}

}  // namespace fa
