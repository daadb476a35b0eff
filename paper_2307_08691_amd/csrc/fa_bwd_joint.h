// The backward pass as ONE grid behind the D pre-pass: the first workgroups take the blocks of keys (dK, dV), heaviest first, the
// others the blocks of query rows (dQ). Nothing passes between the two kinds, so a grid that does not fill the chip takes the time of
// the longer kind instead of the sum, and a larger one has a single half-empty last round instead of two. Results are the bits
// of the two launches of fa_bwd.hip, whose dQ kernel sums D itself and has to end before the dK/dV kernel starts; joint_form says
// which way a problem goes. Included by one source per tile width (they compile side by side).
#pragma once
#include "fa_bwd_work.h"

namespace fa {

template <int D, bool CAUSAL, bool F16, bool DROPOUT, bool PAD, bool MASK, int LOCAL, int DH, int NW, bool SHARED, bool RAGGED, bool SHARE>
__global__ __launch_bounds__(64 * NW) __attribute__((amdgpu_waves_per_eu(D == 128 ? NW / 4 : 2, D == 128 ? NW / 4 : 2))) void
    bwd_joint_kernel(BwdArgs a, unsigned first) {
  typedef DkdvPlan<D, MASK, LOCAL, NW, SHARED> KeyPlan;
  typedef DqPlan<D, MASK, LOCAL, NW> RowPlan;
  __shared__ __attribute__((aligned(1024))) char smem[KeyPlan::SMEM > RowPlan::SMEM ? KeyPlan::SMEM : RowPlan::SMEM];
  if (blockIdx.x < first) {
    // SHARE: all blocks of a share, then those of the next; they go round the XCDs (no room taken for granted) and a share
    // begins beside where the one before it, whose blocks need not divide by eight, ended
    const unsigned part = SHARE ? first / a.shares : first;  // places of one share (a multiple of kXcds)
    const int share = SHARE ? __builtin_amdgcn_readfirstlane(blockIdx.x / part) : 0;
    unsigned place = blockIdx.x - share * part;
    if (SHARE) place = (place & ~(kXcds - 1u)) | ((place - share * a.share_turn) & (kXcds - 1u));
    dkdv_work<D, CAUSAL, F16, DROPOUT, PAD, MASK, LOCAL, DH, NW, SHARED, RAGGED, SHARE>(a, smem, {place, SHARE ? 0 : KeyPlan::SLOTS / 2}, share);
  }
  else dq_work<D, CAUSAL, F16, DROPOUT, PAD, MASK, LOCAL, false, DH, NW, RAGGED>(a, smem, {blockIdx.x - first, RowPlan::SLOTS / 2});
}

template <int D, bool CAUSAL, bool F16, bool DROPOUT, bool PAD, bool MASK, int LOCAL, int DH, int NW, bool SHARED, bool RAGGED, bool SHARE>
static hipError_t launch_joint_as(const BwdArgs& a, hipStream_t st) {
  typedef DkdvPlan<D, MASK, LOCAL, NW, SHARED> KeyPlan;
  typedef DqPlan<D, MASK, LOCAL, NW> RowPlan;
  constexpr int keys = KeyPlan::BC, rows = RowPlan::BR;
  const unsigned first = grid_size(a.p, (a.p.Nk + keys - 1) / keys, a.p.Hkv, SHARE ? 0 : KeyPlan::SLOTS / 2) * (SHARE ? a.shares : 1);
  const unsigned second = grid_size(a.p, (a.p.N + rows - 1) / rows, a.p.Hq, RowPlan::SLOTS / 2);
  hipLaunchKernelGGL((bwd_joint_kernel<D, CAUSAL, F16, DROPOUT, PAD, MASK, LOCAL, DH, NW, SHARED, RAGGED, SHARE>), dim3(first + second), dim3(64 * NW), 0, st, a, first);
  return hipGetLastError();
}

template <int D, bool F16, bool DROPOUT, bool PAD, bool MASK, int DH, int NW, bool SHARED, bool RAGGED, bool SHARE>
static hipError_t launch_joint_rule(const BwdArgs& a, int causal, hipStream_t st) {
  if (causal) return launch_joint_as<D, true, F16, DROPOUT, PAD, MASK, kNoPattern, DH, NW, SHARED, RAGGED, SHARE>(a, st);
  return launch_joint_as<D, false, F16, DROPOUT, PAD, MASK, kNoPattern, DH, NW, SHARED, RAGGED, SHARE>(a, st);
}

template <int D, bool F16, bool RAGGED, bool SHARE>
static hipError_t launch_joint_d(const BwdArgs& a, int causal, hipStream_t st) {
  constexpr int DN = dn_of(D);
  if constexpr (!RAGGED && !SHARE) {
    if (a.p.bmask) return launch_joint_as<D, false, F16, false, false, false, kBlocks, D, 8, false, false, SHARE>(a, st);
    if (a.p.mask) return launch_joint_rule<D, F16, false, false, true, D, 8, false, false, SHARE>(a, causal, st);
  }
  if (windowed(a.p)) return launch_joint_as<D, false, F16, false, false, false, kWindow, D, 8, false, RAGGED, SHARE>(a, st);
  if (a.p.d != D && a.p.d <= DN) return launch_joint_rule<D, F16, false, true, false, DN, 8, false, RAGGED, SHARE>(a, causal, st);
  if (a.p.d != D) return launch_joint_rule<D, F16, false, true, false, D, 8, false, RAGGED, SHARE>(a, causal, st);
  if constexpr (SHARE) {
    if (a.p.drop_thr) return launch_joint_rule<D, F16, true, false, false, D, 8, false, RAGGED, true>(a, causal, st);
    return launch_joint_rule<D, F16, false, false, false, D, 8, false, RAGGED, true>(a, causal, st);
  } else {
    const bool small = joint_small(a, D, causal);
    if (a.p.drop_thr) {
      if constexpr (D == 128) {  // by the rule of the two launches: which form sums a key's rows does not depend on the grid being a joint one
        if (dropout_shared(a.p, causal)) return launch_joint_rule<D, F16, true, false, false, D, 8, true, RAGGED, SHARE>(a, causal, st);
      } else if (small) {
        return launch_joint_rule<D, F16, true, false, false, D, 4, false, RAGGED, SHARE>(a, causal, st);
      }
      return launch_joint_rule<D, F16, true, false, false, D, 8, false, RAGGED, SHARE>(a, causal, st);
    }
    if (small) return launch_joint_rule<D, F16, false, false, false, D, 4, false, RAGGED, SHARE>(a, causal, st);
    return launch_joint_rule<D, F16, false, false, false, D, 8, false, RAGGED, SHARE>(a, causal, st);
  }
}
template <int D, bool F16>
hipError_t launch_joint(const BwdArgs& a, int causal, hipStream_t st) {
  if (hipError_t e = launch_prep<D, F16>(a, st)) return e;
  return a.p.cu_seqlens ? launch_joint_d<D, F16, true, false>(a, causal, st) : launch_joint_d<D, F16, false, false>(a, causal, st);
}
template <int D, bool F16>
hipError_t launch_joint_shares(const BwdArgs& a, int causal, hipStream_t st) {
  if (hipError_t e = launch_prep<D, F16>(a, st)) return e;
  if (hipError_t e = a.p.cu_seqlens ? launch_joint_d<D, F16, true, true>(a, causal, st) : launch_joint_d<D, F16, false, true>(a, causal, st))
    return e;
  return launch_merge_keys(a, st);
}

}  // namespace fa
