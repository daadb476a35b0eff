// Head dimension 256 (Algorithms 1 and 2 of the paper, the same arithmetic as fa_fwd.hip and
// fa_bwd.hip): three kernels of their own, because nothing of the d <= 128 kernels' budget
// carries over. A 32-row (or 32-key) slice of a 256-wide accumulator takes 128 registers, the
// operands another 64 to 128, so a wavefront needs the whole register file of its SIMD (512
// registers, one wavefront per SIMD): workgroups of FOUR wavefronts, 128 query rows (forward,
// dQ) or 128 keys (dK/dV) each, and no second wavefront on the SIMD to run the softmax
// while the first one multiplies. Every kernel is therefore ONE instruction stream in which the vector work of a block
// stands between MFMAs that do not need it (the order of the source, held by scheduling fences), with one barrier
// per block. What bounds such a stream is the number of its instructions (a wavefront alone on its SIMD issues one in
// about five cycles: six beside an MFMA of 32): at N = 8192, causal, 2.7 to 3.6 vector instructions per MFMA, and the matrix pipe is
// busy 52% (forward), 59% (dQ) and 48% (dK/dV) of the cycles at about 2 GHz. Accumulators and operands are placed in the two register
// files by hand (mfma32_agpr and its kin, fa_common.h). Measured (MI355X, bfloat16, 16k tokens in 8 heads, us, plain
// loops around the builtin product -> these): forward N = 2048 causal 179 -> 154, N = 8192 without the mask 1111 -> 944;
// backward 581 -> 521 (25 of them the D pre-pass, now inside the dQ kernel) and 3575 -> 3284.
//
// A 256-wide tile is kept in LDS as two 128-wide halves side by side (columns 0..127 and
// 128..255 of every row), each in the swizzled layout of fa_lds.h, so the operand addressing
// of the d = 128 kernels applies to each half unchanged.
#include "fa_common.h"
#include "fa_kernels.h"
#include "fa_lds.h"

namespace fa {

namespace {

constexpr int kHalf = 128;          // columns of one half tile
constexpr int kRowB = 2 * kHalf;    // its row bytes
template <int ROWS>
using Copier = TileCopier<ROWS, kRowB, 2>;

// lane constants of the operand addressing inside one half tile (fa_lds.h)
struct LaneAddr {
  int zrow;     // 16-byte row operand: (zrow ^ 32 * ks) + row0 * kRowB
  int zcol[2];  // transposing 8-byte reads: (zcol[u] ^ 64 * dt) + 16 * k4 * kRowB
  __device__ __forceinline__ void init(int lane) {
    const int lq = lane & 31, hh = lane >> 5;
    zrow = lq * kRowB + 16 * (hh ^ swz<kRowB>(lq));
    const int p16 = lane & 15, g16 = (lane >> 4) & 1;
#pragma unroll
    for (int u = 0; u < 2; ++u)
      zcol[u] = swz_off<kRowB>(4 * hh + (p16 >> 2) + 8 * u, 2 * g16 + ((p16 & 3) >> 1)) + 8 * (p16 & 1);
  }
};

}  // namespace

// ---------------------------------------------------------------------------------------------
// Forward (Algorithm 1). Wavefront w owns rows 32 w .. 32 w + 31 of a 128-row block; key blocks
// of 64. LDS: three stages of K_j (left | right half, 16 KiB each) and two of V_j.
template <bool CAUSAL, bool F16, bool RAGGED>
__global__ __launch_bounds__(256) __attribute__((amdgpu_waves_per_eu(1, 1))) void fwd256_kernel(FwdArgs a) {
  constexpr int D = 256, BR = 128, BC = 64, KS = D / 16, DT = D / 32;
  constexpr int HALFB = BC * kRowB, TILEB = 2 * HALFB;  // one K_j or V_j: left | right
  constexpr int KSTAGES = 3, V_OFF = KSTAGES * TILEB;     // K_j: three stages, V_j: two (160 KiB in all)
  __shared__ __attribute__((aligned(1024))) char smem[V_OFF + 2 * TILEB];

  const Problem& p = a.p;
  const int tid = threadIdx.x, lane = tid & 63;
  const int w = __builtin_amdgcn_readfirstlane(tid >> 6);
  const int lq = lane & 31, hh = lane >> 5;
  const BlockCoord bc = row_block_coord<CAUSAL, RAGGED>({blockIdx.x, kXcdUnits}, p, BR);
  if (!bc.valid) return;
  const int rowblk = bc.blk;
  const int h = bc.head, s = bc.seq;
  const SeqInfo si = seq_info(p, s);
  const int n = si.n, nk = si.nk, off = nk - n;
  const int i0 = rowblk * BR;
  if (i0 >= n || nk == 0) return;  // (a sequence without keys: see keyless_rows_kernel)
  const int g = __builtin_amdgcn_readfirstlane(h / p.G);  // (else the tile copies keep their addresses per lane)
  const long kstride = (long)p.Hkv * D;
  const __bf16* Kb = a.K + (si.tok0k * p.Hkv + g) * D;
  const __bf16* Vb = a.V + (si.tok0k * p.Hkv + g) * D;

  // Q_i operands in registers (line 4)
  const int prow0 = i0 + 32 * w, row = prow0 + lq;
  const int rowc = row < n ? row : n - 1;  // rows past the end compute on a copy and are never stored
  bf16x8 Qf[KS];
  {
    const __bf16* qp = a.Q + ((si.tok0 + rowc) * p.Hq + h) * D + 8 * hh;
#pragma unroll
    for (int ks = 0; ks < KS; ++ks) Qf[ks] = *(const bf16x8*)(qp + 16 * ks);
  }
  f32x16 O[DT];
#pragma unroll
  for (int dt = 0; dt < DT; ++dt) O[dt] = (f32x16){0};
  float m = -INFINITY, l = 0.f;

  const int ncol_all = (nk + BC - 1) / BC;
  int ncol = ncol_all;
  if (CAUSAL) {
    const int last_pos = (i0 + BR < n ? i0 + BR : n) - 1 + off;
    const int c = last_pos / BC + 1;
    ncol = c < ncol_all ? c : ncol_all;
  }
  if (ncol < 1) ncol = 1;  // (more queries than keys is only allowed without the mask)

  Copier<BC> copier;
  copier.init(kstride, w, lane);
  constexpr int CPT = Copier<BC>::COPIES;  // copies per wavefront and tile
  auto k_stage = [&](int j) { return smem + (j % KSTAGES) * TILEB; };
  auto v_stage = [&](int j) { return smem + V_OFF + (j & 1) * TILEB; };
  // (blocks past the end fetch the last one again, never read, so that the waits can count)
  auto plan = [&](const __bf16* rows, int j) {
    const int jc = j < ncol_all ? j : ncol_all - 1;
    return copier.plan(rows + (long)jc * BC * kstride, nk - 1 - jc * BC);
  };
  static_for<3>([&](auto T) {
    const auto tc = plan(Kb, T.value);
    static_for<CPT>([&](auto Q) { copier.template copy<Q.value>(tc, k_stage(T.value)); });
  });
#pragma unroll
  for (int ks = 0; ks < KS; ++ks) asm volatile("" : "+a"(Qf[ks]));  // (MFMAs take them from there)

  LaneAddr la;
  la.init(lane);
  const float c2 = p.scale_log2e;
  const int lim_row = CAUSAL ? (row + off < nk - 1 ? row + off : nk - 1) : nk - 1;
  f32x16 S[2];           // scores of the current block
  bf16x8 Pp[2][2];       // P of the previous block, rounded: the operand of its O update
  auto k_operand = [&](int st, int i) {  // all of tile 0 (keys 0 .. 31), then of tile 1
    const int ks = i % KS;
    return lds_b128(smem, ((la.zrow + st + (ks >> 3) * HALFB) ^ (32 * (ks & 7))) + (i / KS) * 32 * kRowB);
  };
  auto v_operand = [&](int vst, int i) {
    const int dt = i >> 2, ro = (16 * (i & 3)) * kRowB;
    const int vb = vst + (dt >> 2) * HALFB;
    return lds_tr_pair(smem, ((la.zcol[0] + vb) ^ (64 * (dt & 3))) + ro, ((la.zcol[1] + vb) ^ (64 * (dt & 3))) + ro);
  };
  auto mask = [&](int j) {  // entries above the diagonal and columns past the end
    const int col0 = j * BC;
    if ((CAUSAL && col0 + BC - 1 > prow0 + off) || col0 + BC > nk) {
      mask_past(S, lim_row - col0 - 4 * hh);
    }
  };

  // S_0
  wait_vmem_upto<2 * CPT>();
  lds_barrier();  // K_0 has landed
  {
    const int kst = 0;
    OperandRing ring;
    ring.begin([&](auto I) { return k_operand(kst, I.value); });
    static_for<2 * KS>([&](auto I) {
      constexpr int i = I.value;
      ring.template advance<i, 2 * KS>([&](auto J) { return k_operand(kst, J.value); });
      mfma32_vgpr_ab<F16, i % KS == 0>(S[i / KS], ring.at(I), Qf[i % KS]);
      __builtin_amdgcn_sched_barrier(0);
    });
  }
  settled(S[0], S[1]);
  mask(0);
  m = row_maximum(S);

  // One wavefront per SIMD has to overlap its own matrix and vector work. Iteration j:
  //   O^T += V_{j-1}^T P_{j-1}^T (line 10)     with the exponentials of block j between the MFMAs (line 9)
  //   S_{j+1}^T = K_{j+1} Q_i^T (line 8)       with the tile copies between them
  // in source order, held there by scheduling fences. The exponentials are taken against the reference m as it stands
  // and checked afterwards, as in fwd_kernel (fa_fwd.hip): the row maximum is found only if they outgrew it.
  // One barrier per iteration: it says that K_{j+1} and V_{j-1} have landed everywhere and that everyone has read
  // K_j and V_{j-2}, whose stages this iteration's copies (K_{j+3}, V_j) take.
  auto iteration = [&](int j, auto PV, auto NEXT) {
    constexpr bool pv = decltype(PV)::value, next = decltype(NEXT)::value;
    wait_vmem_upto<CPT>();  // everything but K_{j+2}
    lds_barrier();
    const int vst = V_OFF + ((j + 1) & 1) * TILEB, kst = ((j + 1) % KSTAGES) * TILEB;
    constexpr int NPV = 4 * DT, NS = 2 * KS;
    bf16x8 Pn[2][2];
    float rs0 = 0.f, rs1 = 0.f;
    const float mc = m * c2;
    OperandRing ring;
    if constexpr (pv) ring.begin([&](auto I) { return v_operand(vst, I.value); });
    else if constexpr (next) ring.begin([&](auto I) { return k_operand(kst, I.value); });
    if constexpr (pv) agpr_ready(O);
    u32x4 pw;
    float e0 = 0.f, e1 = 0.f;
    // (a slot consumes the exponential of the slot before it: the result of v_exp_f32 is not ready for the next instruction)
    auto consume = [&](auto E) {
      constexpr int e = decltype(E)::value, kt = e / 16, r = e % 16;
      if constexpr (r & 1) {
        rs1 += e1;
        pw[(r >> 1) & 3] = pack2<F16>(e0, e1);
        if constexpr ((r & 7) == 7) Pn[kt][r >> 3] = __builtin_bit_cast(bf16x8, pw);
      } else {
        rs0 += e0;
      }
    };
    static_for<NPV>([&](auto I) {
      constexpr int i = I.value;
      if constexpr (pv) {
        if constexpr (next)
          ring.template advance<i, NPV + NS>([&](auto J) {
            if constexpr (J.value < NPV) return v_operand(vst, J.value);
            else return k_operand(kst, J.value - NPV);
          });
        else ring.template advance<i, NPV>([&](auto J) { return v_operand(vst, J.value); });
        mfma32_agpr<F16>(O[i >> 2], ring.at(I), Pp[(i >> 1) & 1][i & 1]);
      }
      {
        constexpr int kt = i / 16, r = i % 16;
        float x = __builtin_fmaf(S[kt][r], c2, -mc);
        asm volatile("" : "+v"(x));  // (ties the exponential to this place)
        if constexpr (i > 0) consume(std::integral_constant<int, i - 1>{});
        float& ex = (r & 1) ? e1 : e0;
        ex = fast_exp2(x);
        asm volatile("" : "+v"(ex));
      }
      if constexpr (pv) __builtin_amdgcn_sched_barrier(0);  // keep this order: the two kinds of work alternate
    });
    consume(std::integral_constant<int, NPV - 1>{});
    asm volatile("" ::: "memory");  // (the operands requested for the next stream are not to be requested later)
    if (reference_outgrown<F16>(rs0 + rs1)) {
      const float m_new = fmaxf(m, row_maximum(S));
      const float alpha = fast_exp2((m - m_new) * c2);
      l *= alpha;
      m = m_new;
      if constexpr (pv) {
        agpr_settled(O);
#pragma unroll
        for (int dt = 0; dt < DT; ++dt) {
#pragma unroll
          for (int r = 0; r < 16; ++r) O[dt][r] *= alpha;
          asm volatile("" : "+a"(O[dt]));
        }
      }
      block_exponentials<F16>(S, c2, -m * c2, Pn, rs0, rs1);
    }
    l += rs0 + rs1;
    if constexpr (next) {
      char* vdst = v_stage(j);
      char* kdst = k_stage(j + 3);
      const auto vc = plan(Vb, j), kc = plan(Kb, j + 3);
      static_for<NS>([&](auto I) {
        constexpr int i = I.value;
        if constexpr (pv) ring.template advance<NPV + i, NPV + NS>([&](auto J) { return k_operand(kst, J.value - NPV); });
        else ring.template advance<i, NS>([&](auto J) { return k_operand(kst, J.value); });
        mfma32_vgpr_ab<F16, i % KS == 0>(S[i / KS], ring.at(std::integral_constant<int, pv ? NPV + i : i>{}), Qf[i % KS]);
        if constexpr (i % 2 == 0) {
          constexpr int q = i / 2;
          if constexpr (q < CPT) copier.template copy<q>(vc, vdst);
          else copier.template copy<q - CPT>(kc, kdst);
        }
        __builtin_amdgcn_sched_barrier(0);
      });
      settled(S[0], S[1]);
      mask(j + 1);
    } else {
      const auto vc = plan(Vb, j);
      static_for<CPT>([&](auto Q) { copier.template copy<Q.value>(vc, v_stage(j)); });
    }
#pragma unroll
    for (int kt = 0; kt < 2; ++kt) {
      Pp[kt][0] = Pn[kt][0];
      Pp[kt][1] = Pn[kt][1];
    }
  };
  constexpr std::true_type yes{};
  constexpr std::false_type no{};
  if (ncol > 1) {
    iteration(0, no, yes);
    // (where the loop begins is worth 4% to a wavefront alone on its SIMD, see fa_stream.hip: causal, 1 x 4000, 16 heads, us at 0, 8, .. 56 past
    // a multiple of 64: 134.2, 138.5, 136.3, 138.4, 135.7, 139.2, 135.4, 139.6; grids that fill the chip within 1%)
    asm volatile(".p2align 6");
    for (int j = 1; j < ncol - 1; ++j) iteration(j, yes, yes);
    iteration(ncol - 1, yes, no);
  } else {
    iteration(0, no, no);
  }

  // ---- the last block's O update
  wait_vmem();
  lds_barrier();
  {
    const int vst = V_OFF + ((ncol - 1) & 1) * TILEB;
    OperandRing ring;
    ring.begin([&](auto I) { return v_operand(vst, I.value); });
    agpr_ready(O);
    static_for<4 * DT>([&](auto I) {
      constexpr int i = I.value;
      ring.template advance<i, 4 * DT>([&](auto J) { return v_operand(vst, J.value); });
      mfma32_agpr<F16>(O[i >> 2], ring.at(I), Pp[(i >> 1) & 1][i & 1]);
      __builtin_amdgcn_sched_barrier(0);
    });
  }
  agpr_settled(O);
  lds_barrier();

  // ---- epilogue (lines 12-15): whole rows through LDS, see store_rows_via_lds
  const float lsum = sum_with_partner32(l);
  const float inv = 1.0f / lsum;
  char* stg = smem + w * (32 * kRowB);
  __bf16* op = a.O + ((si.tok0 + prow0) * p.Hq + h) * D;
#pragma unroll
  for (int half = 0; half < 2; ++half)
    store_rows_via_lds<4, F16>(stg, &O[4 * half], inv, op + half * kHalf, (long)p.Hq * D, n - prow0, kHalf, lane);
  if (row < n && hh == 0)
    a.LSE[s * p.lse_seq_stride + h * p.lse_head_stride + (p.cu_seqlens ? si.tok0 : 0) + row] =
        m * p.scale + fast_log2(lsum) * kLn2;
}

template <bool RAGGED>  // a.p.cu_seqlens is set
static hipError_t launch_fwd256_d(const FwdArgs& a, int causal, hipStream_t st) {
  dim3 grid(grid_size(a.p, (a.p.N + 127) / 128, a.p.Hq, kXcdUnits)), block(256);
  if (a.p.f16) {
    if (causal) hipLaunchKernelGGL((fwd256_kernel<true, true, RAGGED>), grid, block, 0, st, a);
    else hipLaunchKernelGGL((fwd256_kernel<false, true, RAGGED>), grid, block, 0, st, a);
  } else {
    if (causal) hipLaunchKernelGGL((fwd256_kernel<true, false, RAGGED>), grid, block, 0, st, a);
    else hipLaunchKernelGGL((fwd256_kernel<false, false, RAGGED>), grid, block, 0, st, a);
  }
  return hipGetLastError();
}
hipError_t launch_fwd256(const FwdArgs& a, int causal, hipStream_t st) {
  return a.p.cu_seqlens ? launch_fwd256_d<true>(a, causal, st) : launch_fwd256_d<false>(a, causal, st);
}

// ---------------------------------------------------------------------------------------------
// dQ (Algorithm 2, lines 10-15 for one row block): the forward kernel's skeleton. Wavefront w owns
// rows 32 w .. of a 128-row block with Q_i, dO_i, L_i, D_i in registers; per key block S^T and
// dP^T = V_j dO_i^T, then P and dS, then dQ_i^T += K_j^T dS^T with K_j^T from transposing reads.
template <bool CAUSAL, bool F16, bool OWN_D, bool RAGGED>
__global__ __launch_bounds__(256) __attribute__((amdgpu_waves_per_eu(1, 1))) void dq256_kernel(BwdArgs a) {
  constexpr int D = 256, BR = 128, BC = 64, KS = D / 16, DT = D / 32;
  constexpr int HALFB = BC * kRowB, TILEB = 2 * HALFB;  // one K_j or V_j: left | right
  constexpr int KSTAGES = 3, V_OFF = KSTAGES * TILEB;     // K_j: three stages, V_j: two (160 KiB in all)
  __shared__ __attribute__((aligned(1024))) char smem[V_OFF + 2 * TILEB];

  const Problem& p = a.p;
  const int tid = threadIdx.x, lane = tid & 63;
  const int w = __builtin_amdgcn_readfirstlane(tid >> 6);
  const int lq = lane & 31, hh = lane >> 5;
  const BlockCoord bc = row_block_coord<CAUSAL, RAGGED>({blockIdx.x, kXcdUnits}, p, BR);
  if (!bc.valid) return;
  const int rowblk = bc.blk;
  const int h = bc.head, s = bc.seq;
  const SeqInfo si = seq_info(p, s);
  const int n = si.n, nk = si.nk, off = nk - n;
  const int i0 = rowblk * BR;
  if (i0 >= n || nk == 0) return;  // (a sequence without keys: see keyless_rows_kernel)
  const int g = __builtin_amdgcn_readfirstlane(h / p.G);  // (else the tile copies keep their addresses per lane)
  const long kstride = (long)p.Hkv * D;
  const __bf16* Kb = a.K + (si.tok0k * p.Hkv + g) * D;
  const __bf16* Vb = a.V + (si.tok0k * p.Hkv + g) * D;

  const int prow0 = i0 + 32 * w, row = prow0 + lq;
  const int rowc = row < n ? row : n - 1;
  bf16x8 Qf[KS], dOf[KS];
  {
    const long qo = ((si.tok0 + rowc) * p.Hq + h) * D + 8 * hh;
#pragma unroll
    for (int ks = 0; ks < KS; ++ks) {
      Qf[ks] = *(const bf16x8*)(a.Q + qo + 16 * ks);
      dOf[ks] = *(const bf16x8*)(a.dO + qo + 16 * ks);
    }
  }
  const long stat = s * p.lse_seq_stride + (long)h * p.lse_head_stride + (p.cu_seqlens ? si.tok0 : 0) + rowc;
  const float Lq = row < n ? a.LSE[stat] * kLog2e : INFINITY;  // rows past the end: P = 0
  f32x16 dQt[DT];
#pragma unroll
  for (int dt = 0; dt < DT; ++dt) dQt[dt] = (f32x16){0};

  const int ncol_all = (nk + BC - 1) / BC;
  int ncol = ncol_all;
  if (CAUSAL) {
    const int last_pos = (i0 + BR < n ? i0 + BR : n) - 1 + off;
    const int c = last_pos / BC + 1;
    ncol = c < ncol_all ? c : ncol_all;
  }
  if (ncol < 1) ncol = 1;

  Copier<BC> copier;
  copier.init(kstride, w, lane);
  constexpr int CPT = Copier<BC>::COPIES;  // copies per wavefront and tile
  auto k_stage = [&](int j) { return smem + (j % KSTAGES) * TILEB; };
  auto v_stage = [&](int j) { return smem + V_OFF + (j & 1) * TILEB; };
  // (blocks past the end fetch the last one again)
  auto plan = [&](const __bf16* rows, int j) {
    const int jc = j < ncol_all ? j : ncol_all - 1;
    return copier.plan(rows + (long)jc * BC * kstride, nk - 1 - jc * BC);
  };
  {
    const auto k0 = plan(Kb, 0), v0 = plan(Vb, 0), k1 = plan(Kb, 1);
    static_for<CPT>([&](auto Q) { copier.template copy<Q.value>(k0, k_stage(0)); });
    static_for<CPT>([&](auto Q) { copier.template copy<Q.value>(v0, v_stage(0)); });
    static_for<CPT>([&](auto Q) { copier.template copy<Q.value>(k1, k_stage(1)); });
  }
  float Dq;
  if constexpr (OWN_D) {  // D_i = rowsum(dO_i o O_i) (line 4), see bwd_dq_kernel in fa_bwd.hip
    const __bf16* op = a.O + ((si.tok0 + rowc) * p.Hq + h) * D + 8 * hh;
    float part = 0.f;
#pragma unroll
    for (int ks = 0; ks < KS; ++ks) {
      const bf16x8 o = *(const bf16x8*)(op + 16 * ks);
      part = dot8<F16>(o, dOf[ks], part);
    }
    Dq = sum_with_partner32(part);
    if (row < n && hh == 0) a.Dvec[stat] = Dq;
  } else {
    Dq = a.Dvec[stat];
  }
#pragma unroll
  for (int ks = 0; ks < KS; ++ks) asm volatile("" : "+a"(Qf[ks]), "+a"(dOf[ks]));  // (MFMAs take them from there)
  touch(Lq);
  touch(Dq);

  LaneAddr la;
  la.init(lane);
  const float c2 = p.scale_log2e;
  const int lim_row = CAUSAL ? (row + off < nk - 1 ? row + off : nk - 1) : nk - 1;
  f32x16 S[2], Sn[2], dP[2];
  bf16x8 dSf[2][2];
  auto row_operand = [&](int st, int i) {  // of K_j or V_j: all of tile 0 (keys 0 .. 31), then of tile 1
    const int ks = i % KS;
    return lds_b128(smem, ((la.zrow + st + (ks >> 3) * HALFB) ^ (32 * (ks & 7))) + (i / KS) * 32 * kRowB);
  };
  auto col_operand = [&](int st, int i) {  // of K_j^T
    const int dt = i >> 2, ro = (16 * (i & 3)) * kRowB, kb = st + (dt >> 2) * HALFB;
    return lds_tr_pair(smem, ((la.zcol[0] + kb) ^ (64 * (dt & 3))) + ro, ((la.zcol[1] + kb) ^ (64 * (dt & 3))) + ro);
  };
  // S_0
  wait_vmem();
  lds_barrier();
  {
    OperandRing ring;
    ring.begin([&](auto I) { return row_operand(0, I.value); });
    static_for<2 * KS>([&](auto I) {
      constexpr int i = I.value;
      ring.template advance<i, 2 * KS>([&](auto J) { return row_operand(0, J.value); });
      mfma32_vgpr_ab<F16, i % KS == 0>(S[i / KS], ring.at(I), Qf[i % KS]);
      __builtin_amdgcn_sched_barrier(0);
    });
  }
  settled(S[0], S[1]);

  // One wavefront per SIMD has to overlap its own matrix and vector work. Iteration j:
  //   dP_j^T = V_j dO_i^T (line 13)           with P_j = exp(S_j - L) (line 11) and the tile copies between the MFMAs
  //   S_{j+1}^T = K_{j+1} Q_i^T (line 10)     with dS_j = P_j o (dP_j - D) (line 14)
  //   dQ_i^T += K_j^T dS_j^T (line 15)        with the registers of S_{j+1} taking the place of S_j's
  // in source order, held there by scheduling fences. One barrier per iteration: V_j and K_{j+1} have landed everywhere, and
  // everyone has read V_{j-1} and K_{j-1}, whose stages this iteration's copies (V_{j+1}, K_{j+2}) take.
  auto iteration = [&](int j, auto NEXT) {
    constexpr bool next = decltype(NEXT)::value;
    if (j > 0) {
      wait_vmem();
      lds_barrier();
    }
    const int kst = (j % KSTAGES) * TILEB, knst = ((j + 1) % KSTAGES) * TILEB, vst = V_OFF + (j & 1) * TILEB;
    constexpr int NA = 2 * KS, NB = next ? 2 * KS : 0, NC = 4 * DT, N = NA + NB + NC;
    auto operand = [&](auto J) {
      constexpr int i = decltype(J)::value;
      if constexpr (i < NA) return row_operand(vst, i);
      else if constexpr (i < NA + NB) return row_operand(knst, i - NA);
      else return col_operand(kst, i - NA - NB);
    };
    const auto vc = plan(Vb, j + 1), kc = plan(Kb, j + 2);
    char *vdst = v_stage(j + 1), *kdst = k_stage(j + 2);
    OperandRing ring;
    ring.begin(operand);
    static_for<NA>([&](auto I) {
      constexpr int i = I.value;
      ring.template advance<i, N>(operand);
      mfma32_vgpr_ab<F16, i % KS == 0>(dP[i / KS], ring.at(I), dOf[i % KS]);
      float x = __builtin_fmaf(S[i >> 4][i & 15], c2, -Lq);
      asm volatile("" : "+v"(x));  // (the empty statements tie the exponential to this place)
      float ex = fast_exp2(x);
      asm volatile("" : "+v"(ex));
      S[i >> 4][i & 15] = ex;
      if constexpr (next && i % 2 == 1) {
        constexpr int q = i / 2;
        if constexpr (q < CPT) copier.template copy<q>(vc, vdst);
        else copier.template copy<q - CPT>(kc, kdst);
      }
      __builtin_amdgcn_sched_barrier(0);
    });
    const int col0 = j * BC;
    asm volatile("" ::: "memory");  // (the operands requested for the next stream are not to be requested later)
    if ((CAUSAL && col0 + BC - 1 > prow0 + off) || (col0 + BC > nk)) {
      asm volatile("; keep this a branch" ::);
#pragma unroll
      for (int kt = 0; kt < 2; ++kt)
#pragma unroll
        for (int r = 0; r < 16; ++r)
          if (col0 + 32 * kt + acc_row(r, hh) > lim_row) S[kt][r] = 0.f;
    }
    if constexpr (!next) settled(dP[0], dP[1]);
    u32x4 pw;
    static_for<2 * KS>([&](auto I) {
      constexpr int i = I.value, kt = i >> 4, r = i & 15;
      if constexpr (next) {
        ring.template advance<NA + i, N>(operand);
        mfma32_vgpr_ab<F16, i % KS == 0>(Sn[i / KS], ring.at(std::integral_constant<int, NA + i>{}), Qf[i % KS]);
      }
      float ds = S[kt][r] * (dP[kt][r] - Dq);
      asm volatile("" : "+v"(ds));
      dP[kt][r] = ds;
      if constexpr (r & 1) pw[(r >> 1) & 3] = pack2<F16>(dP[kt][r - 1], ds);
      if constexpr ((r & 7) == 7) dSf[kt][r >> 3] = __builtin_bit_cast(bf16x8, pw);
      if constexpr (next) __builtin_amdgcn_sched_barrier(0);
    });
    agpr_ready(dQt);
    static_for<NC>([&](auto I) {
      constexpr int i = I.value;
      ring.template advance<NA + NB + i, N>(operand);
      mfma32_agpr<F16>(dQt[i >> 2], ring.at(std::integral_constant<int, NA + NB + i>{}), dSf[(i >> 1) & 1][i & 1]);
      if constexpr (next) asm volatile("v_mov_b32 %0, %1" : "=v"(S[i >> 4][i & 15]) : "v"(Sn[i >> 4][i & 15]));
      __builtin_amdgcn_sched_barrier(0);
    });
  };
  if (ncol > 1) {
    for (int j = 0; j < ncol - 1; ++j) iteration(j, std::true_type{});
    agpr_settled(dQt);  // (where the two paths meet the compiler may move the accumulators)
  }
  iteration(ncol - 1, std::false_type{});

  wait_vmem();
  agpr_settled(dQt);
  lds_barrier();
  char* stg = smem + w * (32 * kRowB);
  __bf16* op = a.dQ + ((si.tok0 + prow0) * p.Hq + h) * D;
#pragma unroll
  for (int half = 0; half < 2; ++half)
    store_rows_via_lds<4, F16>(stg, &dQt[4 * half], p.scale, op + half * kHalf, (long)p.Hq * D, n - prow0, kHalf, lane);
}

// ---------------------------------------------------------------------------------------------
// dK_j, dV_j (Algorithm 2, outer loop over column blocks): a workgroup owns 128 keys of one
// key/value head, wavefront w the 32 keys 32 w .. with their K_j and V_j operands AND the
// dK_j^T, dV_j^T accumulators in registers (384 of them). It walks the query heads of the group
// and, per head, the 32-row tiles Q_i | dO_i (left and right halves, 8 KiB each) that are not
// entirely above the diagonal; L_i and -D_i of the tile's rows sit beside them in LDS.
template <bool CAUSAL, bool F16, bool RAGGED>
__global__ __launch_bounds__(256) __attribute__((amdgpu_waves_per_eu(1, 1))) void dkdv256_kernel(BwdArgs a) {
  constexpr int D = 256, BC = 128, BR = 32, KS = D / 16, DT = D / 32;
  constexpr int HALFB = BR * kRowB, STAGEB = 4 * HALFB;  // Q left | Q right | dO left | dO right
  constexpr int RING = 3;  // tiles in LDS
  constexpr int LS_OFF = RING * STAGEB, DV_OFF = LS_OFF + RING * BR * 4, SMEM = DV_OFF + RING * BR * 4;
  __shared__ __attribute__((aligned(1024))) char smem[SMEM < 4 * 32 * kRowB ? 4 * 32 * kRowB : SMEM];

  const Problem& p = a.p;
  const int tid = threadIdx.x, lane = tid & 63;
  const int w = __builtin_amdgcn_readfirstlane(tid >> 6);
  const int lq = lane & 31, hh = lane >> 5;
  const BlockCoord bc = key_block_coord<CAUSAL, RAGGED>({blockIdx.x, kXcdUnits}, p, BC);
  if (!bc.valid) return;
  const int g = bc.head, s = bc.seq;
  const SeqInfo si = seq_info(p, s);
  const int n = si.n, nk = si.nk, off = nk - n;
  const int j0 = bc.blk * BC;
  if (j0 >= nk) return;
  const long qstride = (long)p.Hq * D;
  const float c2 = p.scale_log2e;
  const int nrt = (n + BR - 1) / BR;
  int i_first = CAUSAL && j0 > off ? (j0 - off) / BR : 0;  // row tiles entirely above the diagonal are skipped
  if (i_first > nrt) i_first = nrt;
  const int per_head = nrt - i_first, T = per_head * p.G;
  const long stat_base = s * p.lse_seq_stride + (p.cu_seqlens ? si.tok0 : 0);

  // K_j, V_j operands of this lane's key (line 6): registers for the whole kernel
  const int key0 = j0 + 32 * w, key = key0 + lq;
  const bool key_ok = key < nk;
  bf16x8 Kf[KS], Vf[KS];
  {
    const long ko = ((si.tok0k + (key_ok ? key : nk - 1)) * p.Hkv + g) * D + 8 * hh;
#pragma unroll
    for (int ks = 0; ks < KS; ++ks) {
      Kf[ks] = *(const bf16x8*)(a.K + ko + 16 * ks);
      Vf[ks] = *(const bf16x8*)(a.V + ko + 16 * ks);
    }
  }
  f32x16 dKt[DT], dVt[DT];
#pragma unroll
  for (int dt = 0; dt < DT; ++dt) dKt[dt] = dVt[dt] = (f32x16){0};

  // tile t = (head g G + t / per_head, row tile i_first + t % per_head)
  float lraw = 0.f, draw = 0.f;
  bool stat_ok = false;
  // (tiles are requested in order: the head and row tile of the next request are carried along; past the last tile it is
  // requested again, never read)
  Copier<BR> copier;
  copier.init(qstride, w, lane);
  constexpr int CPT = Copier<BR>::COPIES;  // copies per wavefront of Q_i, as many of dO_i
  int next_hq = g * p.G, next_it = i_first, next_t = 0;
  struct Request {
    typename Copier<BR>::Plan q, o;
    char* dst;
  };
  auto request = [&]() {  // the next tile's copies (to be issued) and its statistics (on their way)
    const int hq = next_hq, it = next_it;
    Request r;
    r.dst = smem + (next_t % RING) * STAGEB;
    if (next_t < T - 1 && ++next_it == nrt) {
      next_it = i_first;
      ++next_hq;
    }
    ++next_t;
    const long first = ((si.tok0 + (long)it * BR) * p.Hq + hq) * D;
    r.q = copier.plan(a.Q + first, n - 1 - it * BR);
    r.o = copier.plan(a.dO + first, n - 1 - it * BR);
    if (tid < BR) {
      const int row = it * BR + tid;
      stat_ok = row < n;
      const long si_ = stat_base + (long)hq * p.lse_head_stride + (stat_ok ? row : n - 1);
      lraw = a.LSE[si_];
      draw = a.Dvec[si_];
    }
    return r;
  };
  auto commit_stats = [&](int t) {
    touch(lraw);
    touch(draw);
    if (tid < BR) {
      // L in the exponent's base; rows past the end get L = +inf so that P = 0. D is stored
      // negated: it is the initial value of the dP accumulator (line 14).
      *(float*)(smem + LS_OFF + ((t % RING) * BR + tid) * 4) = stat_ok ? lraw * kLog2e : INFINITY;
      *(float*)(smem + DV_OFF + ((t % RING) * BR + tid) * 4) = stat_ok ? -draw : 0.f;
    }
  };
  LaneAddr la;
  la.init(lane);
  f32x16 S, dP;
  f32x4 Lv[4];
  bf16x8 Pf[2], dSf[2];
  auto row_operand = [&](int st, int i) { return lds_b128(smem, (la.zrow + st + (i >> 3) * HALFB) ^ (32 * (i & 7))); };
  auto col_operand = [&](int st, int i) {  // dt = i / 2, contraction half i % 2
    const int dt = i >> 1, qoff = st + (dt >> 2) * HALFB + 16 * (i & 1) * kRowB;
    return lds_tr_pair(smem, (la.zcol[0] + qoff) ^ (64 * (dt & 3)), (la.zcol[1] + qoff) ^ (64 * (dt & 3)));
  };
  auto load_stats = [&](int t) {  // dP starts from -D_i (line 14)
#pragma unroll
    for (int r4 = 0; r4 < 4; ++r4) {
      const f32x4 Dn = *(const f32x4*)(smem + DV_OFF + ((t % RING) * BR + 8 * r4 + 4 * hh) * 4);
      Lv[r4] = *(const f32x4*)(smem + LS_OFF + ((t % RING) * BR + 8 * r4 + 4 * hh) * 4);
#pragma unroll
      for (int u = 0; u < 4; ++u) dP[4 * r4 + u] = Dn[u];
    }
  };
  if (T > 0) {
#pragma unroll
    for (int t = 0; t < 2; ++t) {
      const Request r = request();
      static_for<CPT>([&](auto Q) { copier.template copy<Q.value>(r.q, r.dst); });
      static_for<CPT>([&](auto Q) { copier.template copy<Q.value>(r.o, r.dst + 2 * HALFB); });
      commit_stats(t);
    }
#pragma unroll
    for (int ks = 0; ks < KS; ++ks) {
      touch(Kf[ks]);
      touch(Vf[ks]);
    }
    wait_vmem();
    lds_barrier();
    {
      OperandRing ring;
      ring.begin([&](auto I) { return row_operand(0, I.value); });
      static_for<KS>([&](auto I) {
        constexpr int i = I.value;
        ring.template advance<i, KS>([&](auto J) { return row_operand(0, J.value); });
        mfma32_vgpr<F16, i == 0>(S, ring.at(I), Kf[i]);
        __builtin_amdgcn_sched_barrier(0);
      });
    }
    load_stats(0);
    settled(S);
  }

  // One wavefront per SIMD has to overlap its own matrix and vector work. Iteration t:
  //   dP_t - D = dO_i V_j^T - D (line 13)   with P_t = exp(S_t - L) (line 11) between the MFMAs
  //   dV_j^T += dO_i^T P_t (line 12)        with dS_t = P_t o (dP_t - D) (line 14)
  //   S_{t+1} = Q_{i'} K_j^T (line 10)      with the copies of tile t + 2
  //   dK_j^T += Q_i^T dS_t (line 16)        with the statistics of tile t + 1
  // in source order, held there by scheduling fences. One barrier per iteration: tile t + 1 has landed everywhere, and
  // everyone has read tile t - 1, whose place this iteration's copies take.
  int cur_it = i_first;  // row tile of tile t
  auto iteration = [&](int t, auto NEXT) {
    constexpr bool next = decltype(NEXT)::value;
    if (t > 0) {
      wait_vmem();
      commit_stats(t + 1);
      lds_barrier();
    }
    const int st = (t % RING) * STAGEB, nst = ((t + 1) % RING) * STAGEB;
    const int r0 = cur_it * BR;  // first query row of the tile
    if (++cur_it == nrt) cur_it = i_first;
    constexpr int NA = KS, NV = 2 * DT, NB = next ? KS : 0, NK = 2 * DT, N = NA + NV + NB + NK;
    auto operand = [&](auto J) {
      constexpr int i = decltype(J)::value;
      if constexpr (i < NA) return row_operand(st + 2 * HALFB, i);
      else if constexpr (i < NA + NV) return col_operand(st + 2 * HALFB, i - NA);
      else if constexpr (i < NA + NV + NB) return row_operand(nst, i - NA - NV);
      else return col_operand(st, i - NA - NV - NB);
    };
    OperandRing ring;
    ring.begin(operand);
    static_for<NA>([&](auto I) {
      constexpr int i = I.value;
      ring.template advance<i, N>(operand);
      mfma32_vgpr<F16, false>(dP, ring.at(I), Vf[i]);
      float x = __builtin_fmaf(S[i], c2, -Lv[i >> 2][i & 3]);
      asm volatile("" : "+v"(x));  // (the empty statements tie the exponential to this place)
      float ex = fast_exp2(x);
      asm volatile("" : "+v"(ex));
      S[i] = ex;
      __builtin_amdgcn_sched_barrier(0);
    });
    asm volatile("" ::: "memory");  // (the operands requested for the next stream are not to be requested later)
    if ((CAUSAL && key0 + 31 > r0 + off) || j0 + BC > nk) {
      asm volatile("; keep this a branch" ::);
      // visible: key < nk and (causal) key <= r0 + off + row of the tile, row = acc_row(r, hh)
      const int kc = key_ok ? (CAUSAL ? key - (r0 + off) - 4 * hh : -1) : 0x7fffffff;
#pragma unroll
      for (int r = 0; r < 16; ++r) S[r] = kc <= acc_row(r, 0) ? S[r] : 0.f;
    }
    Pf[0] = pack8<F16>(S, 0);
    Pf[1] = pack8<F16>(S, 1);
    asm volatile("" : "+v"(Pf[0]), "+v"(Pf[1]));
    agpr_ready(dVt);
    u32x4 pw;
    static_for<NV>([&](auto I) {
      constexpr int i = I.value;
      ring.template advance<NA + i, N>(operand);
      mfma32_agpr<F16>(dVt[i >> 1], ring.at(std::integral_constant<int, NA + i>{}), Pf[i & 1]);
      // (the first entries of dP after the MFMAs above have had time to finish)
      if constexpr (i % 2 == 1) {
        static_for<2>([&](auto U) {
          constexpr int r = i - 1 + U.value;
          float ds = dP[r] * S[r];
          asm volatile("" : "+v"(ds));
          dP[r] = ds;
          if constexpr (r & 1) pw[(r >> 1) & 3] = pack2<F16>(dP[r - 1], ds);
          if constexpr ((r & 7) == 7) dSf[r >> 3] = __builtin_bit_cast(bf16x8, pw);
        });
      }
      __builtin_amdgcn_sched_barrier(0);
    });
    if constexpr (next) {
      const Request r = request();
      static_for<NB>([&](auto I) {
        constexpr int i = I.value;
        ring.template advance<NA + NV + i, N>(operand);
        mfma32_vgpr<F16, i == 0>(S, ring.at(std::integral_constant<int, NA + NV + i>{}), Kf[i]);
        if constexpr (i % 2 == 0) {
          constexpr int q = i / 2;
          if constexpr (q < CPT) copier.template copy<q>(r.q, r.dst);
          else copier.template copy<q - CPT>(r.o, r.dst + 2 * HALFB);
        }
        __builtin_amdgcn_sched_barrier(0);
      });
    }
    agpr_ready(dKt);
    static_for<NK>([&](auto I) {
      constexpr int i = I.value;
      ring.template advance<NA + NV + NB + i, N>(operand);
      mfma32_agpr<F16>(dKt[i >> 1], ring.at(std::integral_constant<int, NA + NV + NB + i>{}), dSf[i & 1]);
      if constexpr (next && i == NK - 4) load_stats(t + 1);
      __builtin_amdgcn_sched_barrier(0);
    });
  };
  for (int t = 0; t < T - 1; ++t) iteration(t, std::true_type{});
  if (T > 0) iteration(T - 1, std::false_type{});

  wait_vmem();
  agpr_settled(dKt);
  agpr_settled(dVt);
  lds_barrier();
  // ---- write dK_j, dV_j (line 18); dK carries the scaling
  char* stg = smem + w * (32 * kRowB);
  const long kvoff = ((si.tok0k + key0) * p.Hkv + g) * D;
#pragma unroll
  for (int half = 0; half < 2; ++half) {
    store_rows_via_lds<4, F16>(stg, &dKt[4 * half], p.scale, a.dK + kvoff + half * kHalf, (long)p.Hkv * D, nk - key0, kHalf, lane);
    store_rows_via_lds<4, F16>(stg, &dVt[4 * half], 1.f, a.dV + kvoff + half * kHalf, (long)p.Hkv * D, nk - key0, kHalf, lane);
  }
}

template <bool RAGGED>
static hipError_t launch_dkdv256(const BwdArgs& a, int causal, hipStream_t st) {
  dim3 grid(grid_size(a.p, (a.p.Nk + 127) / 128, a.p.Hkv, kXcdUnits)), block(256);
  if (a.p.f16) {
    if (causal) hipLaunchKernelGGL((dkdv256_kernel<true, true, RAGGED>), grid, block, 0, st, a);
    else hipLaunchKernelGGL((dkdv256_kernel<false, true, RAGGED>), grid, block, 0, st, a);
  } else {
    if (causal) hipLaunchKernelGGL((dkdv256_kernel<true, false, RAGGED>), grid, block, 0, st, a);
    else hipLaunchKernelGGL((dkdv256_kernel<false, false, RAGGED>), grid, block, 0, st, a);
  }
  return hipGetLastError();
}
template <bool F16, bool OWN_D, bool RAGGED>
static hipError_t launch_dq256(const BwdArgs& a, int causal, hipStream_t st) {
  dim3 grid(grid_size(a.p, (a.p.N + 127) / 128, a.p.Hq, kXcdUnits)), block(256);
  if (causal) hipLaunchKernelGGL((dq256_kernel<true, F16, OWN_D, RAGGED>), grid, block, 0, st, a);
  else hipLaunchKernelGGL((dq256_kernel<false, F16, OWN_D, RAGGED>), grid, block, 0, st, a);
  return hipGetLastError();
}
template <bool RAGGED>
static hipError_t launch_bwd256_whole(const BwdArgs& a, int causal, hipStream_t st) {
  // (the dQ kernel sums D on the way, the dK/dV kernel reads it)
  if (hipError_t e = a.p.f16 ? launch_dq256<true, true, RAGGED>(a, causal, st) : launch_dq256<false, true, RAGGED>(a, causal, st)) return e;
  return launch_dkdv256<RAGGED>(a, causal, st);
}
hipError_t launch_bwd256(const BwdArgs& a, int causal, int stages, hipStream_t st) {
  if (stages == 7) return a.p.cu_seqlens ? launch_bwd256_whole<true>(a, causal, st) : launch_bwd256_whole<false>(a, causal, st);
  if (a.p.cu_seqlens || a.p.f16) return hipErrorInvalidValue;  // (one stage or two: fa_bwd_stages, dense batches in bfloat16)
  if (stages & 2)
    if (hipError_t e = launch_dkdv256<false>(a, causal, st)) return e;
  if (stages & 4) return launch_dq256<false, false, false>(a, causal, st);
  return hipSuccess;
}

}  // namespace fa
