// Forward pass (Algorithm 1 of the paper) for grids that do not fill the chip: d = 64 and 128, dense or packed, no options.
//
// On such a grid the time is the chain of the longest workgroup, and fwd_kernel (fa_fwd.hip) makes that chain long: 256
// rows, two wavefronts per SIMD that take turns with the matrix pipe, every block a matrix phase AND a vector phase
// (1.25 us per block of 64 keys at d = 128). Here a workgroup has FOUR wavefronts and 128 rows, one wavefront per SIMD
// (two workgroups fit on a compute unit), and a wavefront is one instruction stream in which the softmax of a block
// stands between products that do not need it, as in the d = 256 kernels (0.93 us per block; bound by the number of
// instructions, one in about five cycles from one wavefront, and by the copies, 35 cycles each). The arithmetic is
// that of fwd_kernel operation by operation, so the results are the same bits and the size of the grid may choose the form.
// Measured (MI355X, bfloat16, causal, us from fwd_kernel to this one): d = 128: 1 x 1531, 32 heads on 8: 36.3 -> 31.2;
// 1 x 1024, 16 heads: 25.5 -> 19.9; 1 x 4096, 8 heads: 78.8 -> 63.9; d = 64: 1 x 8192, 8 heads: 130 -> 98;
// 1 x 128, 2 heads, no mask: 5.9 -> 4.7. On full grids the two wavefronts per SIMD of fwd_kernel are the faster form
// (2 x 8192, 16 heads of 128: 449 there, 484 here): see stream_form in fa_fwd.hip.
#include "fa_common.h"
#include "fa_kernels.h"
#include "fa_lds.h"

namespace fa {

template <int D, bool CAUSAL, bool F16, bool RAGGED>
__global__ __launch_bounds__(256) __attribute__((amdgpu_waves_per_eu(2, 2))) void fwd_stream_kernel(FwdArgs a) {
  constexpr int BR = 128, BC = 64, KS = D / 16, DT = D / 32, ROWB = 2 * D;
  constexpr int TILEB = BC * ROWB;
  constexpr int KSTAGES = 3, V_OFF = KSTAGES * TILEB;  // K_j: three stages, V_j: two (80 KiB at d = 128)
  __shared__ __attribute__((aligned(1024))) char smem[V_OFF + 2 * TILEB];

  const Problem& p = a.p;
  const int tid = threadIdx.x, lane = tid & 63;
  const int w = __builtin_amdgcn_readfirstlane(tid >> 6);
  const int lq = lane & 31, hh = lane >> 5;
  const BlockCoord bc = row_block_coord<CAUSAL, RAGGED>({blockIdx.x, 2 * kXcdUnits}, p, BR);
  if (!bc.valid) return;
  const int h = bc.head, s = bc.seq;
  const SeqInfo si = seq_info(p, s);
  const int n = si.n, nk = si.nk, off = nk - n;
  const int i0 = bc.blk * BR;
  if (i0 >= n || nk == 0) return;  // (a sequence without keys: see keyless_rows_kernel)
  const int g = __builtin_amdgcn_readfirstlane(h / p.G);
  const long kstride = (long)p.Hkv * D;
  const __bf16* Kb = a.K + (si.tok0k * p.Hkv + g) * D;
  const __bf16* Vb = a.V + (si.tok0k * p.Hkv + g) * D;
  const int prow0 = i0 + 32 * w, row = prow0 + lq;
  const int rowc = row < n ? row : n - 1;  // rows past the end compute on a copy and are never stored
  const int ncol_all = (nk + BC - 1) / BC;
  int ncol = ncol_all, ncolw = ncol_all;  // blocks that the workgroup, that this wavefront visits
  if (CAUSAL) {
    const int c = ((i0 + BR < n ? i0 + BR : n) - 1 + off) / BC + 1, cw = (prow0 + 31 + off) / BC + 1;
    ncol = c < ncol_all ? c : ncol_all;
    ncolw = cw < ncol ? cw : ncol;
    // A packed sequence may hold fewer keys than queries, which the host cannot see; its first rows then see none. All wavefronts
    // visit a block all the same: they share the barriers and the copies, and each has to make as many of both.
    if (RAGGED && ncol < 1) ncol = 1;
    if (RAGGED && ncolw < 1) ncolw = 1;
  }

  typedef TileCopier<BC, ROWB> Copier;
  Copier copier;
  copier.init(kstride, w, lane);
  constexpr int CPT = Copier::COPIES;  // copies per wavefront and tile
  // The next blocks of K and V to be copied: where their rows begin, the last valid row counted from there, and where they
  // go. (Blocks past the end fetch the last one again, never read, so that the waits can count. Carried along: an
  // instruction saved is five cycles.)
  struct Next {
    const __bf16* base;
    int last;
  };
  Next next_k = {Kb, nk - 1}, next_v = {Vb, nk - 1};
  const long step = (long)BC * kstride;
  auto advance = [&](Next& x) {
    const bool more = x.last >= BC;
    x.base += more ? step : 0;
    x.last -= more ? BC : 0;
  };
  int kslot = 0, vslot = 0;  // stage that the next K (V) block goes to
  auto copy_k = [&]() {
    const auto t = copier.plan(next_k.base, next_k.last);
    static_for<CPT>([&](auto Q) { copier.template copy<Q.value>(t, smem + kslot); });
    kslot = kslot == (KSTAGES - 1) * TILEB ? 0 : kslot + TILEB;
    advance(next_k);
  };
  auto copy_v = [&]() {
    const auto t = copier.plan(next_v.base, next_v.last);
    static_for<CPT>([&](auto Q) { copier.template copy<Q.value>(t, smem + V_OFF + vslot); });
    vslot ^= TILEB;
    advance(next_v);
  };
  copy_k();
  char* const qst = smem + V_OFF + w * (32 * ROWB);  // (no V tile is on its way yet)
  rows_request<D>(qst, a.Q + (si.tok0 * p.Hq + h) * D, (long)p.Hq * D, prow0, n - 1, lane);
  copy_k();
  copy_k();
  f32x16 O[DT];
#pragma unroll
  for (int dt = 0; dt < DT; ++dt) O[dt] = (f32x16){0};
  float m, l = 0.f;

  const int zrow = lq * ROWB + 16 * (hh ^ swz<ROWB>(lq));
  const int p16 = lane & 15, g16 = (lane >> 4) & 1;
  int zcol[2];
#pragma unroll
  for (int u = 0; u < 2; ++u)
    zcol[u] = swz_off<ROWB>(4 * hh + (p16 >> 2) + 8 * u, 2 * g16 + ((p16 & 3) >> 1)) + 8 * (p16 & 1);
  const float c2 = p.scale_log2e;
  const int lim_row = CAUSAL ? (row + off < nk - 1 ? row + off : nk - 1) : nk - 1;
  f32x16 S[2];      // scores of the current block
  bf16x8 Pp[2][2];  // P of the previous block, rounded: the operand of its O update
  auto k_operand = [&](int st, int i) {  // all of tile 0 (keys 0 .. 31), then of tile 1
    return lds_b128(smem, ((zrow + st) ^ (32 * (i % KS))) + (i / KS) * 32 * ROWB);
  };
  auto v_operand = [&](int st, int i) {
    const int dt = i >> 2, ro = (16 * (i & 3)) * ROWB;
    return lds_tr_pair(smem, ((zcol[0] + st) ^ (64 * dt)) + ro, ((zcol[1] + st) ^ (64 * dt)) + ro);
  };
  auto mask = [&](int j) {  // entries above the diagonal and columns past the end
    const int col0 = j * BC;
    if ((CAUSAL && col0 + BC - 1 > prow0 + off) || col0 + BC > nk) {
      asm volatile("; keep this a branch: the mask costs two instructions per element" ::);
      mask_past(S, lim_row - col0 - 4 * hh);
    }
  };
  wait_vmem_upto<2 * CPT>();
  bf16x8 Qf[KS];
  row_operands<D>(Qf, qst, lane);
  lds_barrier();  // K_0 has landed
  {
    OperandRing ring;
    ring.begin([&](auto I) { return k_operand(0, I.value); });
    static_for<2 * KS>([&](auto I) {
      constexpr int i = I.value;
      ring.template advance<i, 2 * KS>([&](auto J) { return k_operand(0, J.value); });
      mfma32_vgpr<F16, i % KS == 0>(S[i / KS], ring.at(I), Qf[i % KS]);
      __builtin_amdgcn_sched_barrier(0);
    });
  }
  settled(S[0], S[1]);
  mask(0);
  m = row_maximum(S);

  // Iteration j:
  //   O^T += V_{j-1}^T P_{j-1}^T (line 10)     with the exponentials of block j between the MFMAs (line 9)
  //   S_{j+1}^T = K_{j+1} Q_i^T (line 8)       with the copies of K_{j+3} between them (those of V_j stand at the start)
  // in source order, held there by scheduling fences. One barrier per iteration: K_{j+1} and V_{j-1} have landed everywhere,
  // and everyone has read K_j and V_{j-2}, whose stages K_{j+3} and V_j take. The exponentials are taken against the
  // reference m as it stands and checked afterwards, see fwd_kernel.
  int kst = TILEB;  // stage of K_{j+1}
  auto iteration = [&](int j, auto PV, auto NEXT) {
    constexpr bool pv = decltype(PV)::value, next = decltype(NEXT)::value;
    wait_vmem_upto<CPT>();  // everything but K_{j+2}
    lds_barrier();
    const int vst = V_OFF + (vslot ^ TILEB);  // (vslot: where V_j goes)
    constexpr int NPV = 4 * DT, NS = 2 * KS, EPS = 32 / NPV;  // exponentials beside an MFMA of the O update
    constexpr int N = (pv ? NPV : 0) + (next ? NS : 0), S0 = pv ? NPV : 0;
    auto operand = [&](auto J) {
      constexpr int i = decltype(J)::value;
      if constexpr (i < S0) return v_operand(vst, i);
      else return k_operand(kst, i - S0);
    };
    bf16x8 Pn[2][2];
    float rs0 = 0.f, rs1 = 0.f;
    const float mc = m * c2;
    OperandRing ring;
    if constexpr (N > 0) ring.begin(operand);
    copy_v();  // (as early as its stage is free: it has this iteration to arrive)
    u32x4 pw;
    float ex[2][EPS];
    auto consume = [&](auto SLOT) {
      static_for<EPS>([&](auto U) {
        constexpr int e = decltype(SLOT)::value * EPS + U.value, kt = e / 16, r = e % 16;
        float(&x)[EPS] = ex[decltype(SLOT)::value & 1];
        if constexpr (r & 1) {
          rs1 += x[U.value];
          pw[(r >> 1) & 3] = pack2<F16>(x[U.value - 1], x[U.value]);
          if constexpr ((r & 7) == 7) Pn[kt][r >> 3] = __builtin_bit_cast(bf16x8, pw);
        } else {
          rs0 += x[U.value];
        }
      });
    };
    static_for<NPV>([&](auto I) {
      constexpr int i = I.value;
      float x[EPS];
      static_for<EPS>([&](auto U) {
        constexpr int e = i * EPS + U.value;
        x[U.value] = __builtin_fmaf(S[e / 16][e % 16], c2, -mc);
        asm volatile("" : "+v"(x[U.value]));  // (ties the exponential to this place)
      });
      if constexpr (i > 0) consume(std::integral_constant<int, i - 1>{});
      static_for<EPS>([&](auto U) {
        ex[i & 1][U.value] = fast_exp2(x[U.value]);
        asm volatile("" : "+v"(ex[i & 1][U.value]));
      });
      if constexpr (pv) {
        ring.template advance<i, N>(operand);
        mfma32_vgpr<F16, false>(O[i >> 2], ring.at(I), Pp[(i >> 1) & 1][i & 1]);
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
        settled(O);
#pragma unroll
        for (int dt = 0; dt < DT; ++dt)
#pragma unroll
          for (int r = 0; r < 16; ++r) O[dt][r] *= alpha;
      }
      block_exponentials<F16>(S, c2, -m * c2, Pn, rs0, rs1);
    }
    l += rs0 + rs1;
    if constexpr (next) {
      const auto kc = copier.plan(next_k.base, next_k.last);
      static_for<NS>([&](auto I) {
        constexpr int i = I.value;
        ring.template advance<S0 + i, N>(operand);
        mfma32_vgpr<F16, i % KS == 0>(S[i / KS], ring.at(std::integral_constant<int, S0 + i>{}), Qf[i % KS]);
        if constexpr (i % 2 == 0 && i / 2 < CPT) copier.template copy<i / 2>(kc, smem + kslot);
        __builtin_amdgcn_sched_barrier(0);
      });
      kslot = kst;  // (K_{j+4} takes the place of K_{j+1})
      kst = kst == (KSTAGES - 1) * TILEB ? 0 : kst + TILEB;
      advance(next_k);
      settled(S[0], S[1]);
      mask(j + 1);
    } else if (j + 1 < ncol) {
      copy_k();  // (other wavefronts go on)
    }
#pragma unroll
    for (int kt = 0; kt < 2; ++kt) {
      Pp[kt][0] = Pn[kt][0];
      Pp[kt][1] = Pn[kt][1];
    }
  };
  constexpr std::true_type yes{};
  constexpr std::false_type no{};
  if (ncolw > 1) {
    iteration(0, no, yes);
    // Where the loop begins: a wavefront alone on its SIMD waits for instructions that straddle a fetch, and the compiler lays the loop
    // wherever the code before it ends. Bytes past a multiple of 64, the best of sixteen places (MI355X, us, at the worst and here:
    // causal, d = 64, 1 x 1292, 4 heads 19.0 and 18.4, 2 x 2112 27.6 and 26.6; 2 heads of 128, 3119: 52.2 and 50.4; no mask, d = 64, 1 x 1777, 8
    // heads 24.9 and 22.6; grids that fill the chip: no difference). Under a condition of its own: the loop is then entered without a
    // test, which the compiler would lay in between, longer or shorter by instantiation (packed batches, causal, d = 128, 6 of up to 68
    // on 2377: 42.3 so and 41.3 here), and who does not loop does not go through the filling (1 x 128, 2 heads of 64: 4.56 and 4.50).
    if (ncolw > 2) {
      if constexpr (D == 64 && !CAUSAL) asm volatile(".p2align 6\n.rept 7\ns_nop 0\n.endr");
      else if constexpr (D == 64) asm volatile(".p2align 6\n.rept 1\ns_nop 0\n.endr");
      else if constexpr (!CAUSAL) asm volatile(".p2align 6\n.rept 6\ns_nop 0\n.endr");
      else asm volatile(".p2align 6\n.rept 2\ns_nop 0\n.endr");
      for (int j = 1; j < ncolw - 1; ++j) iteration(j, yes, yes);
    }
    iteration(ncolw - 1, yes, no);
  } else {
    iteration(0, no, no);
  }
  // ---- the last block's O update; a wavefront whose rows see fewer blocks than the workgroup's last ones then only keeps up
  wait_vmem();
  lds_barrier();
  const int vlast = V_OFF + (vslot ^ TILEB);
  if (ncolw < ncol) {
    copy_v();
    copy_k();
  }
  {
    const int vst = vlast;
    OperandRing ring;
    ring.begin([&](auto I) { return v_operand(vst, I.value); });
    static_for<4 * DT>([&](auto I) {
      constexpr int i = I.value;
      ring.template advance<i, 4 * DT>([&](auto J) { return v_operand(vst, J.value); });
      mfma32_vgpr<F16, false>(O[i >> 2], ring.at(I), Pp[(i >> 1) & 1][i & 1]);
      __builtin_amdgcn_sched_barrier(0);
    });
  }
  settled(O);
  for (int j = ncolw + 1; j <= ncol; ++j) {
    wait_vmem_upto<CPT>();
    lds_barrier();
    if (j < ncol) {
      copy_v();
      copy_k();
    }
  }
  wait_vmem();
  lds_barrier();  // the tiles have been read by everyone, no copy is on its way

  // ---- epilogue (lines 12-15)
  const float lsum = sum_with_partner32(l);
  const float inv = 1.0f / lsum;
  char* stg = smem + w * (32 * ROWB);
  __bf16* op = a.O + ((si.tok0 + prow0) * p.Hq + h) * D;
  store_rows_via_lds<DT, F16>(stg, O, inv, op, (long)p.Hq * D, n - prow0, D, lane);
  if (row < n && hh == 0)
    a.LSE[s * p.lse_seq_stride + h * p.lse_head_stride + (p.cu_seqlens ? si.tok0 : 0) + row] =
        m * p.scale + fast_log2(lsum) * kLn2;
}

template <int D, bool F16, bool RAGGED>
static hipError_t launch_stream_d(const FwdArgs& a, int causal, hipStream_t st) {
  const dim3 grid(grid_size(a.p, (a.p.N + 127) / 128, a.p.Hq, 2 * kXcdUnits)), block(256);
  if (causal) hipLaunchKernelGGL((fwd_stream_kernel<D, true, F16, RAGGED>), grid, block, 0, st, a);
  else hipLaunchKernelGGL((fwd_stream_kernel<D, false, F16, RAGGED>), grid, block, 0, st, a);
  return hipGetLastError();
}
hipError_t launch_fwd_stream(const FwdArgs& a, int d, int causal, hipStream_t st) {
  const bool r = a.p.cu_seqlens != nullptr;
  if (a.p.f16) {
    if (d == 64) return r ? launch_stream_d<64, true, true>(a, causal, st) : launch_stream_d<64, true, false>(a, causal, st);
    return r ? launch_stream_d<128, true, true>(a, causal, st) : launch_stream_d<128, true, false>(a, causal, st);
  }
  if (d == 64) return r ? launch_stream_d<64, false, true>(a, causal, st) : launch_stream_d<64, false, false>(a, causal, st);
  return r ? launch_stream_d<128, false, true>(a, causal, st) : launch_stream_d<128, false, false>(a, causal, st);
}

}  // namespace fa
