"""The rules that choose a kernel, on the CPU (launches.py)."""
import shutil
import subprocess
import types

import pytest

import forms

from launches import P, cross_bwd, dropout_bwd, launches, mask_bwd, varlen_bwd, varlen_cross_bwd
from paper_2307_08691_amd import binding


@pytest.mark.parametrize("nseq,nq,nk,Hq,Hkv,d", [(16, 4096, 128, 16, 16, 128), (16, 4096, 128, 16, 16, 64), (6, 382, 8030, 4, 4, 128),
                                                 (15, 387, 6909, 1, 1, 128), (3, 700, 900, 8, 4, 64), (40, 2000, 60, 8, 8, 128)])
@pytest.mark.parametrize("f16", [False, True])
def test_packed_batches_of_two_lengths_count_their_keys(nseq, nq, nk, Hq, Hkv, d, f16):
    """The blocks of keys of a packed batch are counted by its keys, not by its queries: under four rounds of them on the compute units
    the backward is one grid (joint_form), whatever the number of queries."""
    packed, more = launches([varlen_cross_bwd(nseq, nseq * nq, nseq * nk, nq, nk, Hq, Hkv, d, False, f16),
                             varlen_cross_bwd(nseq, nseq * nq * 64, nseq * nk, nq * 64, nk, Hq, Hkv, d, False, f16)])
    assert (nk / 256 + 0.5) * nseq * Hkv / 256 < 4
    for kernels in (packed, more):
        assert ["keyless" in kernels[0][0], "bwd_prep" in kernels[1][0], "bwd_joint" in kernels[2][0]] == [True] * 3 and len(kernels) == 3


@pytest.mark.parametrize("d", [64, 128])
def test_many_rounds_of_keys_are_two_launches_for_few_queries_too(d):
    few, many = launches([varlen_cross_bwd(64, 64 * 16, 64 * 8192, 16, 8192, 8, 8, d), varlen_cross_bwd(64, 64 * 8192, 64 * 8192, 8192, 8192, 8, 8, d)])
    for kernels in (few, many):
        assert [k[0].split("<")[0].split()[-1] for k in kernels[1:]] == ["bwd_dq_kernel", "bwd_dkdv_kernel"]


def form(kernels):
    return "one grid" if any("bwd_joint" in k[0] for k in kernels) else "two launches"


@pytest.mark.parametrize("call,want", [
    (cross_bwd(32, 16, 2, 44, 3127, 64), "two launches"), (cross_bwd(18, 32, 16, 103, 585, 64), "two launches"),
    (cross_bwd(18, 32, 16, 631, 631, 64, f16=True), "two launches"), (mask_bwd(2, 8, 8, 199, 8152, 128, f16=True), "two launches"),
    (mask_bwd(1, 32, 8, 123, 7714, 128), "two launches"), (cross_bwd(12, 8, 8, 900, 900, 80), "one grid"),
    (mask_bwd(10, 32, 16, 934, 54, 64), "one grid"), (cross_bwd(2, 1, 1, 2304, 2304, 128), "one grid"), (cross_bwd(1, 8, 4, 448, 448, 64, True), "one grid"),
    (cross_bwd(27, 16, 16, 600, 600, 128), "one grid"), (cross_bwd(25, 32, 32, 268, 268, 64), "two launches"),
    (dropout_bwd(4, 16, 16, 1777, 1777, 64, f16=True), "one grid"),
    (cross_bwd(16, 16, 16, 1024, 1024, 128), "two launches"), (cross_bwd(8, 32, 32, 2048, 2048, 64), "two launches")])
def test_the_backward_is_one_grid_where_that_ends_sooner(call, want):
    """Shapes whose two forms were measured (joint_sooner, joint_form): rests of rounds alone do not make one grid the sooner form."""
    assert form(launches([call])[0]) == want


@pytest.mark.parametrize("lens,Hq,Hkv,d", [([3000], 8, 1, 64), ([700, 1, 0, 233], 8, 1, 128), ([1500] * 8, 32, 4, 64), ([321, 100], 8, 1, 128),
                                           ([128] * 16, 32, 8, 128), ([1201], 4, 1, 128), ([4000, 12], 16, 4, 96)])
def test_packed_batches_get_the_workspace_that_they_use(lens, Hq, Hkv, d):
    """The workspace that the binding allocates for a packed batch, which knows the longest sequence, is as good as the larger one of
    fa_varlen_bwd_workspace_bytes, which does not."""
    x = types.SimpleNamespace(Tq=sum(lens), Hq=Hq, Hkv=Hkv, d=d)
    used, bound = binding._packed_bwd_bytes(x, max(lens)), binding.fa_varlen_bwd_workspace_bytes(x.Tq, Hq, Hkv, d)
    assert used <= bound
    a, b = launches([varlen_bwd(len(lens), x.Tq, max(lens), Hq, Hkv, d, w) for w in (used, bound)])
    assert a == b
    assert any("merge" in k[0] for k in a) <= (used > 4 * x.Tq * Hq + 255)


def test_every_backward_kernel_is_launched_by_a_problem_that_runs_on_the_gpu():
    """The problems of forms.py reach every instantiation of the two-launch kernels, of the one grid and of the short form. Not counted:
    those that only single stages take (fa_bwd_stages: a dQ kernel that is given D; 128-key blocks at d = 128 under the causal
    rule) and the grids with shares (test_shares_of_a_block_of_keys)."""
    if not shutil.which("nm"):
        pytest.skip("lists the library's kernels with nm")
    names = subprocess.run(["nm", "-DC", binding.LIB_PATH], capture_output=True, text=True, check=True).stdout.splitlines()
    kernels = {n.split("fa::", 1)[1].rsplit("(", 1)[0] for n in names if " V " in n and "fa::" in n}
    args = lambda k: k[k.index("<") + 1:-1].split(", ")
    want = {k for k in kernels if k.startswith(("bwd_dkdv_kernel", "bwd_short_kernel")) or (k.startswith("bwd_dq_kernel") and args(k)[7] == "true") or
            (k.startswith("bwd_joint_kernel") and args(k)[11] == "false")}
    want -= {k for k in want if k.startswith("bwd_dkdv_kernel<128, true, false") and args(k)[8] == "4"}
    assert len(want) > 300
    reached = launches([forms.backward_call(*c, f16) for c in forms.cases() for f16 in (False, True)])
    assert not want - {k[0] for call in reached for k in call}


@pytest.mark.parametrize("B,Hkv,d,cap,num_splits", [(33, 8, 64, 512, 1), (33, 8, 128, 512, 1), (11, 8, 128, 1536, 3), (21, 8, 64, 1280, 2)])
@pytest.mark.parametrize("f16", [False, True])
def test_many_short_caches_share_a_compute_unit(B, Hkv, d, cap, num_splits, f16):
    """The problems of test_many_short_paged_caches take the form of two workgroups on a compute unit."""
    for causal in (False, True):
        kernels = launches([("fa_kvcache_fwd", [P] * 8 + [1 << 40, B, Hkv, Hkv, 1, cap, d, 64, cap // 64, 0.1, causal, num_splits, 0, f16])])[0]
        assert kernels[0][0] == f"fwd_decode_kernel<{d}, {str(causal).lower()}, {str(f16).lower()}, true>"
