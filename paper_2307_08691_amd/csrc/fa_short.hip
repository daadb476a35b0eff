// Backward pass (Algorithm 2 of the paper) of short sequences in ONE kernel: d = 64, up to 512 tokens, dense or packed, no options.
//
// The two kernels of fa_bwd.hip each read Q, K, V, dO, form S and dP and take the exponentials (seven products where five
// do) because dQ summed across workgroups would need atomics. Up to 512 keys ONE workgroup holds all of a sequence's dK and dV in
// its accumulators, so nothing is summed across workgroups: it visits the rows in tiles of 32, every wavefront forms P
// and dS of its own 32 (KW = 1) or 2 x 32 (KW = 2) keys, adds to its dK_j, dV_j (lines 12, 16) and leaves dS in LDS, where
// one phase later two wavefronts, in turn, form the tile's dQ_i = dS K over all keys (line 15; K is in LDS for the whole kernel).
// Measured (MI355X, bfloat16, 32 x 512, 32 heads, causal, us of the backward): 270 -> 215; 64 x 256: 216 -> 171; 128 x 128: 194 -> 133.
// What bounds it: waiting (at 32 x 512 the matrix pipe is busy 18% of the time, LDS 23%, and the wavefronts wait 43% of theirs). Half
// of the time passed with the row tiles left out (a workgroup's K, V, O, dO arrive before its first tile, and beyond 128 tokens there
// is no second workgroup on the compute unit to fill that time); the rest is the chain of a phase, LDS reads, MFMAs, exponentials,
// barrier (the exponentials left out: 2 us less, dQ left out: 42).
// The arithmetic is that of the two kernels operation by operation and in their order, so the results are the same bits
// and the size of the grid may choose the form (short_form).
#include "fa_common.h"
#include "fa_kernels.h"
#include "fa_lds.h"

namespace fa {

// KW: 32-key pieces per wavefront, NW: wavefronts (keys: up to 32 NW KW; wavefront w owns the pieces w, w + NW, so that under
// the mask the pieces that a row tile sees are spread over the SIMDs).
template <int KW, int NW>
struct ShortPlan {
  static constexpr int D = 64, ROWB = 2 * D, KEYS = 32 * NW * KW, RING = 3;
  static constexpr int TILEB = 32 * ROWB, SLOTB = 2 * TILEB;   // a slot of the ring: Q_i | dO_i
  static constexpr int DS_OFF = KEYS * ROWB;                   // dS^T: [key][2 x 32 rows], the tiles take the halves in turn
  static constexpr int RING_OFF = DS_OFF + KEYS * ROWB;
  static constexpr int STG_OFF = RING_OFF + RING * SLOTB;      // two 32 x 32 pieces of dQ on their way out
  static constexpr int L_OFF = STG_OFF + 2 * 2048;
  static constexpr int STATS = KW == 2 ? 512 : 2048;           // rows (over the group's query heads) whose L, D fit
  // where O_i and dO_i pass through at the start: dS^T's place, and for 256 keys (one workgroup per compute unit either way) more
  static constexpr int EXTRA_OFF = L_OFF + 8 * STATS, EXTRA = KW == 1 && NW == 8 ? NW * TILEB : 0;
  static constexpr int SMEM = EXTRA_OFF + EXTRA;
};

// (one block a pair: the pairs go round the XCDs by themselves, and a short step's time is the chain that its workgroup starts with)
constexpr int kAnyNumber = 0x7fffffff;

template <int KW, int NW, bool CAUSAL, bool F16>
__global__ __launch_bounds__(64 * NW) __attribute__((amdgpu_waves_per_eu(2, 2))) void bwd_short_kernel(BwdArgs a) {
  typedef ShortPlan<KW, NW> Plan;
  constexpr int D = Plan::D, ROWB = Plan::ROWB, KS = D / 16, DT = D / 32, RING = Plan::RING;
  static_assert(Plan::SMEM <= 160 * 1024, "LDS of one compute unit");
  __shared__ __attribute__((aligned(1024))) char smem[Plan::SMEM];
  float* const Ls = (float*)(smem + Plan::L_OFF);
  float* const Ds = Ls + Plan::STATS;

  const Problem& p = a.p;
  const int tid = threadIdx.x, lane = tid & 63;
  const int w = __builtin_amdgcn_readfirstlane(tid >> 6);
  const int lq = lane & 31, hh = lane >> 5;
  const BlockCoord bc = block_coord<false, true>({blockIdx.x, kAnyNumber}, 1, p.Hkv, p.nseq);  // (from the last pair to the first: see launch_bwd_d)
  if (!bc.valid) return;
  const int g = bc.head, s = bc.seq;
  const SeqInfo si = seq_info(p, s);
  const int n = si.n < p.N ? si.n : p.N;  // rows = keys (a packed batch: never more than the bound that the caller states)
  if (n <= 0) return;
  const int pieces = (n + 31) / 32, nrt = (n + 63) / 64;  // of 32 keys; row tiles of 64, each visited as two of 32
  const int rows64 = 64 * nrt;
  const long qstride = (long)p.Hq * D, kstride = (long)p.Hkv * D;
  const float c2 = p.scale_log2e;

  // The order of the visits is that of the dK/dV kernel: row tiles of 64, in each the query heads of the group.
  struct Visit {
    int r0, hi;  // first row, query head inside the group
  };
  const int T = 2 * nrt * p.G;
  auto next = [&](const Visit& v) {
    Visit x = v;
    if (x.r0 & 32) {
      x.r0 -= 32;
      if (++x.hi == p.G) {
        x.hi = 0;
        x.r0 += 64;
      }
    } else {
      x.r0 += 32;
    }
    return x;
  };

  // ---- copies: a Q_i | dO_i tile is eight pieces of 1 KiB, one (NW = 8) or two per wavefront
  constexpr int CP = 8 / NW;
  auto copy_tile = [&](const Visit& v, int slot) {
    int ln = lane;  // (recomputed for every tile instead of held in registers)
    asm volatile("" : "+v"(ln));
    const int crow = 8 * (w & 3) + ln / 8, c = 8 * ((ln % 8) ^ swz<ROWB>(crow));
    const int r = v.r0 + crow < n ? v.r0 + crow : n - 1;
    const long o = ((si.tok0 + r) * p.Hq + g * p.G + v.hi) * D + c;
    char* dst = smem + Plan::RING_OFF + slot * Plan::SLOTB + (w & 3) * 1024;
    if (NW == 4 || w < 4) dma16(a.Q + o, dst);
    if (NW == 4 || w >= 4) dma16(a.dO + o, dst + Plan::TILEB);
  };

  // ---- K into LDS (keys up to the end of the last piece; past the end of the sequence they repeat its last)
  {
    const __bf16* Kb = a.K + (si.tok0k * p.Hkv + g) * D;
    for (int rb = 8 * w; rb < 32 * pieces; rb += 8 * NW) {
      const int r = rb + lane / 8, rc = r < n ? r : n - 1;
      dma16(Kb + rc * kstride + 8 * ((lane % 8) ^ swz<ROWB>(r)), smem + rb * ROWB);
    }
  }
  Visit ld = {0, 0};  // next tile to copy
  copy_tile(ld, 0);
  ld = next(ld);
  copy_tile(ld, 1);
  ld = next(ld);
  // ---- V operands of the wavefront's keys: registers for the whole kernel
  bf16x8 Vf[KW][KS];
#pragma unroll
  for (int u = 0; u < KW; ++u) {
    const int key = 32 * (NW * u + w) + lq;
    const __bf16* vp = a.V + ((si.tok0k + (key < n ? key : n - 1)) * p.Hkv + g) * D + 8 * hh;
#pragma unroll
    for (int ks = 0; ks < KS; ++ks) Vf[u][ks] = *(const bf16x8*)(vp + 16 * ks);
  }
  // ---- L and D = rowsum(dO o O) (line 4) of all rows, as the dQ kernel sums it: a lane takes half a row
  // (O_i, and dO_i where there is room, come through a piece of the idle dS^T area as whole rows: straight into registers a
  // request touches 16 bytes of each of 32 rows twice: 32 x 512 causal 224 -> 215 us, 128 x 128 144 -> 133)
  constexpr bool BOTH = KW == 2 || Plan::EXTRA;
  const char* const stage = smem + Plan::DS_OFF + w * (KW * Plan::TILEB);
  const char* const stage2 = KW == 2 ? stage + Plan::TILEB : smem + Plan::EXTRA_OFF + w * Plan::TILEB;
  const int orow = lq * ROWB + 16 * (hh ^ swz<ROWB>(lq));
  for (int q = w; q < p.G * (rows64 / 32); q += NW) {
    const int hi = q / (rows64 / 32), row = 32 * (q - hi * (rows64 / 32)) + lq, rowc = row < n ? row : n - 1;
    const int h = g * p.G + hi;
    const long o = ((si.tok0 + rowc) * p.Hq + h) * D + 8 * hh;
    const float lse = a.LSE[s * p.lse_seq_stride + (long)h * p.lse_head_stride + (p.cu_seqlens ? si.tok0 : 0) + rowc];
    bf16x8 ov[KS], gv[KS];
    asm volatile("s_waitcnt lgkmcnt(0)" ::: "memory");  // (the rows before these have been read)
#pragma unroll
    for (int u = 0; u < 4; ++u) {
      const int sr = 8 * u + lane / 8, r = row - lq + sr < n ? row - lq + sr : n - 1;
      const long so = ((si.tok0 + r) * p.Hq + h) * D + 8 * ((lane % 8) ^ swz<ROWB>(sr));
      dma16(a.O + so, stage + 1024 * u);
      if (BOTH) dma16(a.dO + so, stage2 + 1024 * u);
    }
    if (!BOTH) {
#pragma unroll
      for (int ks = 0; ks < KS; ++ks) gv[ks] = *(const bf16x8*)(a.dO + o + 16 * ks);
    }
    wait_vmem();
#pragma unroll
    for (int ks = 0; ks < KS; ++ks) {
      ov[ks] = lds_b128(stage, orow ^ (32 * ks));
      if (BOTH) gv[ks] = lds_b128(stage2, orow ^ (32 * ks));
    }
    float part = 0.f;
#pragma unroll
    for (int ks = 0; ks < KS; ++ks) part = dot8<F16>(ov[ks], gv[ks], part);
    const float dsum = sum_with_partner32(part);
    if (hh == 0) {
      Ls[hi * rows64 + row] = row < n ? lse * kLog2e : INFINITY;  // rows past the end: P = 0
      Ds[hi * rows64 + row] = row < n ? -dsum : 0.f;
    }
  }
#pragma unroll
  for (int u = 0; u < KW; ++u)
#pragma unroll
    for (int ks = 0; ks < KS; ++ks) touch(Vf[u][ks]);
  wait_vmem();
  lds_barrier();

  // ---- lane constants of the LDS addressing (see the dK/dV kernel)
  const int zrow = lq * ROWB + 16 * (hh ^ swz<ROWB>(lq));
  const int p16 = lane & 15, g16 = (lane >> 4) & 1;
  int zcol[2];
#pragma unroll
  for (int u = 0; u < 2; ++u)
    zcol[u] = swz_off<ROWB>(4 * hh + (p16 >> 2) + 8 * u, 2 * g16 + ((p16 & 3) >> 1)) + 8 * (p16 & 1);
  const int zds = Plan::DS_OFF + (32 * w + lq) * ROWB + 16 * swz<ROWB>(lq) + 8 * hh;  // this lane's key in dS^T; chunk c at ^ 16 c

  f32x16 dKt[KW][DT], dVt[KW][DT];
#pragma unroll
  for (int u = 0; u < KW; ++u)
#pragma unroll
    for (int dt = 0; dt < DT; ++dt) dKt[u][dt] = dVt[u][dt] = (f32x16){0};
  bf16x8 Pf[2], dSf[2];

  // P and dS of the wavefront's piece U on the tile `v` in ring slot at byte `qb` (lines 10, 11, 13, 14); dS also to LDS
  auto scores = [&](const Visit& v, int qb, auto U) {
    constexpr int u = decltype(U)::value;
    const int piece = NW * u + w;
    const int zq = zrow + qb, zk = zrow + 32 * piece * ROWB;
    const int st = v.hi * rows64 + v.r0 + 4 * hh;
    f32x16 S = (f32x16){0}, dP;
#pragma unroll
    for (int r4 = 0; r4 < 4; ++r4) {
      const f32x4 Dn = *(const f32x4*)(Ds + st + 8 * r4);
#pragma unroll
      for (int e = 0; e < 4; ++e) dP[4 * r4 + e] = Dn[e];
    }
    mfma_stream<2 * KS, 4, 2>(
        [&](int i) {
          const int x = 32 * (i % KS);
          if (i < KS) return OperandPair{lds_b128(smem, zq ^ x), lds_b128(smem, zk ^ x)};
          const bf16x8 o = lds_b128(smem, (zq ^ x) + Plan::TILEB);
          return OperandPair{o, o};
        },
        [&](int i, const OperandPair& o) {
          if (i < KS) S = mfma32<F16>(o.a, o.b, S);
          else dP = mfma32<F16>(o.a, Vf[u][i % KS], dP);
        });
#pragma unroll
    for (int r4 = 0; r4 < 4; ++r4) {
      const f32x4 Lv = *(const f32x4*)(Ls + st + 8 * r4);
#pragma unroll
      for (int e = 0; e < 4; ++e) S[4 * r4 + e] = fast_exp2(__builtin_fmaf(S[4 * r4 + e], c2, -Lv[e]));
    }
    if ((CAUSAL && 32 * piece == v.r0) || 32 * piece + 32 > n) {  // on the diagonal, at the end of the sequence
      asm volatile("; keep this a branch: the mask costs two instructions per element" ::);
      const int key = 32 * piece + lq;
      const int kc = key < n ? (CAUSAL ? key - v.r0 - 4 * hh : -1) : 0x7fffffff;
#pragma unroll
      for (int r = 0; r < 16; ++r) S[r] = kc <= acc_row(r, 0) ? S[r] : 0.f;
    }
#pragma unroll
    for (int r = 0; r < 16; ++r) dP[r] *= S[r];
    const int zd = (zds + 32 * NW * u * ROWB) ^ (2 * (v.r0 & 32));
#pragma unroll
    for (int s2 = 0; s2 < 2; ++s2) {
      Pf[s2] = pack8<F16>(S, s2);
      dSf[s2] = pack8<F16>(dP, s2);
      const u32x4 x = __builtin_bit_cast(u32x4, dSf[s2]);
      *(u32x2*)(smem + (zd ^ (32 * s2))) = (u32x2){x[0], x[1]};
      *(u32x2*)(smem + (zd ^ (32 * s2 + 16))) = (u32x2){x[2], x[3]};
    }
  };
  // dV_j^T += dO_i^T P (line 12), dK_j^T += Q_i^T dS (line 16)
  auto update = [&](int qb, auto U) {
    constexpr int u = decltype(U)::value;
    const int zc0 = zcol[0] + qb, zc1 = zcol[1] + qb;
    mfma_stream<4 * DT, 8, 2>(
        [&](int i) {
          const int dt = i >> 2, ro = 16 * ((i >> 1) & 1) * ROWB + (i & 1) * Plan::TILEB;
          return lds_tr_pair(smem, (zc0 ^ (64 * dt)) + ro, (zc1 ^ (64 * dt)) + ro);
        },
        [&](int i, bf16x8 x) {
          const int dt = i >> 2, s2 = (i >> 1) & 1;
          if (i & 1) dVt[u][dt] = mfma32<F16>(x, Pf[s2], dVt[u][dt]);
          else dKt[u][dt] = mfma32<F16>(x, dSf[s2], dKt[u][dt]);
        });
  };
  // dQ_i^T = K^T dS^T (line 15) of the tile `v`, columns 32 dt .. 32 dt + 31, over all keys that it sees; scaled and stored
  auto dq_piece = [&](const Visit& v, int dt) {
    int np = pieces;
    if (CAUSAL && v.r0 / 32 + 1 < np) np = v.r0 / 32 + 1;
    const int half = 2 * (v.r0 & 32);
    const int k0 = zcol[0] ^ (64 * dt), k1 = zcol[1] ^ (64 * dt);
    const int d0 = (zcol[0] ^ half) + Plan::DS_OFF, d1 = (zcol[1] ^ half) + Plan::DS_OFF;
    __builtin_amdgcn_s_setprio(3);  // (the others wait for it at the barrier: 32 x 512 causal 233 -> 224 us)
    f32x16 acc = (f32x16){0};
    bf16x8 k[3][2], d[3][2];  // operands of three pieces: requested two pieces (four MFMAs) ahead
    auto fetch = [&](int i, int q) {
      const int o = 32 * (q < np ? q : np - 1) * ROWB;
#pragma unroll
      for (int s2 = 0; s2 < 2; ++s2) {
        const int ro = o + 16 * s2 * ROWB;
        k[i][s2] = lds_tr_pair(smem, k0 + ro, k1 + ro);
        d[i][s2] = lds_tr_pair(smem, d0 + ro, d1 + ro);
      }
    };
    auto piece = [&](int i, int q) {
      fetch((i + 2) % 3, q + 2);
      __builtin_amdgcn_sched_barrier(0);
      acc = mfma32<F16>(k[i][0], d[i][0], acc);
      acc = mfma32<F16>(k[i][1], d[i][1], acc);
      __builtin_amdgcn_sched_barrier(0);
    };
    fetch(0, 0);
    fetch(1, 1);
    int q = 0;
    for (; q + 3 <= np; q += 3) {
      piece(0, q);
      piece(1, q + 1);
      piece(2, q + 2);
    }
    if (q < np) piece(0, q);
    if (q + 1 < np) piece(1, q + 1);
    __builtin_amdgcn_s_setprio(0);
    __bf16* op = a.dQ + ((si.tok0 + v.r0) * p.Hq + g * p.G + v.hi) * D + 32 * dt;
    int ln = lane;  // recomputed here: nothing of the staging addresses is to live across the main loop
    asm volatile("" : "+v"(ln));
    store_rows_via_lds<1, F16>(smem + Plan::STG_OFF + dt * 2048, &acc, p.scale, op, qstride, n - v.r0, 32, ln);
  };

  // ---- phase t: dQ of tile t - 1 (two wavefronts, in turn), P, dS of tile t and its dK, dV update; one barrier at the end. It
  // orders what goes through LDS: dS of tile t takes the half that dQ of tile t - 2 was read from in phase t - 1; tile
  // t + 2 takes the ring slot that tile t - 1 was read from in phase t - 1, and has phases t and t + 1 to arrive.
  Visit cur = {0, 0}, prev = {0, 0};
  int slot = 0;
  for (int t = 0; t <= T; ++t) {
    if (t > 0 && prev.r0 < n) {
      // (under the mask the last wavefronts: they have the fewest pieces to see)
      const int dt = CAUSAL ? NW - 1 - w : (w - 2 * (t - 1)) & (NW - 1);
      if (dt < DT) dq_piece(prev, dt);
    }
    if (t == T) break;
    // (the stores of dQ are older than this copy, so that the wait below covers them)
    if (t + 2 < T) {
      copy_tile(ld, slot == 0 ? RING - 1 : slot - 1);
      ld = next(ld);
    }
    const int seen = CAUSAL && cur.r0 / 32 + 1 < pieces ? cur.r0 / 32 + 1 : pieces;  // pieces that the tile's rows see
    if (cur.r0 < n) {
      const int qb = Plan::RING_OFF + slot * Plan::SLOTB;
      static_for<KW>([&](auto U) {
        if (NW * U.value + w < seen) {
          __builtin_amdgcn_sched_barrier(0);
          scores(cur, qb, U);
          __builtin_amdgcn_sched_barrier(0);
          update(qb, U);
          __builtin_amdgcn_sched_barrier(0);
        }
      });
    }
    if (t + 2 < T) wait_vmem_upto<CP>();
    else wait_vmem();
    lds_barrier();
    prev = cur;
    cur = next(cur);
    slot = slot == RING - 1 ? 0 : slot + 1;
  }
  lds_barrier();  // dS has been read by everyone

  // ---- write dK_j, dV_j (line 18); dK carries the scaling
  char* stg = smem + Plan::DS_OFF + w * (32 * ROWB);
#pragma unroll
  for (int u = 0; u < KW; ++u) {
    const int key0 = 32 * (NW * u + w);
    if (key0 < n) {
      const long o = ((si.tok0k + key0) * p.Hkv + g) * D;
      store_tiles_via_lds<DT, F16>(stg, dKt[u], p.scale, a.dK + o, kstride, n - key0, D, lane);
      store_tiles_via_lds<DT, F16>(stg, dVt[u], 1.f, a.dV + o, kstride, n - key0, D, lane);
    }
  }
}

template <int KW, int NW>
static hipError_t launch_short(const BwdArgs& a, int causal, hipStream_t st) {
  const dim3 grid(grid_size(1, a.p.Hkv * a.p.nseq, kAnyNumber)), block(64 * NW);
  if (a.p.f16) {
    if (causal) hipLaunchKernelGGL((bwd_short_kernel<KW, NW, true, true>), grid, block, 0, st, a);
    else hipLaunchKernelGGL((bwd_short_kernel<KW, NW, false, true>), grid, block, 0, st, a);
  } else {
    if (causal) hipLaunchKernelGGL((bwd_short_kernel<KW, NW, true, false>), grid, block, 0, st, a);
    else hipLaunchKernelGGL((bwd_short_kernel<KW, NW, false, false>), grid, block, 0, st, a);
  }
  return hipGetLastError();
}

// Whether the whole backward is one kernel (the head dimension is 64 and there are no options: the caller has looked): up to
// 512 tokens, as many rows as the tables of L and D hold, and a grid on which it was measured to win. A workgroup
// stands for a whole (sequence, key/value head) pair, so few pairs leave compute units idle, and beyond 256 tokens, where its chain
// is long, a last round of workgroups that is mostly empty costs a whole one; the two kernels of fa_bwd.hip cut a pair into more
// workgroups. (MI355X, bfloat16, us of the backward from the two kernels to this one; 16 heads unless stated.)
//  * no more pairs than compute units, no shared heads, up to 192 tokens, or 256 under the mask: one short launch instead of two
//    (1 x 128: 20.9 -> 18.1, 16 x 192: 24.5 -> 20.9, 4 x 256 causal 22.7 -> 19.5, without the mask 21.4 -> 22.7).
//  * up to 256 tokens: from 192 pairs on (64 x 128: 49.7 -> 35.7; 64 x 256, 32 heads on 4: 160 -> 120; 17 x 256: 272 pairs, 49.7 ->
//    46.4; 32 x 256, 32 heads on 4: 128 pairs, 101 -> 111).
//  * beyond: rounds of 256 that are three quarters full (32 x 512, 32 heads, causal 270 -> 215; 12 x 512: 192 pairs, 58.7 -> 50.2;
//    24 x 512: 384, 102 -> 94; 33 x 512: 528, 143 -> 141; 4 x 512: 64, 32.4 -> 44.3), without the mask, where the chains are longer
//    still and there is more than one round, seven eighths (32 x 512, 32 heads: 330 -> 288; 24 x 512: 384, 125 -> 127).
bool bwd_short_form(const Problem& p, int causal) {
  if (p.N > 512 || p.cu_seqlens_k || (!p.cu_seqlens && p.N != p.Nk)) return false;
  const long pairs = (long)p.Hkv * p.nseq, rows = (long)p.G * 64 * ((p.N + 63) / 64);
  if (rows > (p.N > 256 ? ShortPlan<2, 8>::STATS : ShortPlan<1, 8>::STATS)) return false;
  if (p.G == 1 && pairs <= 256 && p.N <= (causal ? 256 : 192)) return true;
  if (p.N <= 256) return pairs >= 192;
  const long rounds = (pairs + 255) / 256;
  return 8 * pairs >= (causal || rounds == 1 ? 6 : 7) * 256 * rounds;
}
hipError_t launch_bwd_short(const BwdArgs& a, int causal, hipStream_t st) {
  if (a.p.N <= 128) return launch_short<1, 4>(a, causal, st);
  if (a.p.N <= 256) return launch_short<1, 8>(a, causal, st);
  return launch_short<2, 8>(a, causal, st);
}

}  // namespace fa
