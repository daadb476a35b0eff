"""GPU parity with dropout on P: fa_dropout_fwd / fa_dropout_bwd against the float64 oracle, which
regenerates the same keep mask from the same (seed, head, query, key) function. The mask decision
is integer arithmetic on both sides. The outputs carry the factor 1 / (1 - p), so what is asserted is
the yardstick clause: no worse than a bf16 implementation of the standard algorithm with the same
keep mask that materialises S and P (parity_util.judge with standard=False)."""
import numpy as np
import pytest

from paper_2307_08691_amd import binding, inputs
from oracle import attention_oracle as orc

pytestmark = pytest.mark.gpu

torch = pytest.importorskip("torch")
import parity_util as pu  # noqa: E402


def run(prob, p_drop, seed):
    Q, K, V, dO = (pu.to_gpu(x, prob.dtype) for x in (prob.Q, prob.K, prob.V, prob.dO))
    O, L = binding.fa_dropout_fwd(Q, K, V, prob.scale, prob.causal, p_drop, seed)
    dQ, dK, dV = binding.fa_dropout_bwd(Q, K, V, O, dO, L, prob.scale, prob.causal, p_drop, seed)
    torch.cuda.synchronize()
    return dict(O=O, LSE=L, dQ=dQ, dK=dK, dV=dV)


def keep_masks(seed, p_drop, Hq):
    """keep_of(sequence, head, nq, nk) for parity_util.reference_batch, from the oracle's generator."""
    thr = orc.dropout_threshold(p_drop)
    return (lambda s, h, nq, nk: torch.from_numpy(orc.dropout_keep(seed, s * Hq + h, nq, nk, thr)).cuda()), 256.0 / (256.0 - thr)


def check_dropout(prob, p_drop, seed):
    got = run(prob, p_drop, seed)
    widen = orc.widen_f16 if prob.dtype == "f16" else orc.widen_bf16
    Q, K, V, dO = (widen(x) for x in (prob.Q, prob.K, prob.V, prob.dO))
    exp = {}
    exp["O"], exp["LSE"] = orc.attention_forward_dropout(Q, K, V, prob.scale, prob.causal, p_drop, seed)
    exp["dQ"], exp["dK"], exp["dV"] = orc.attention_backward_dropout(Q, K, V, dO, prob.scale, prob.causal, p_drop, seed)
    keep_of, rp = keep_masks(seed, p_drop, prob.Hq)
    ref = pu.reference_batch(*(pu.to_gpu(x, prob.dtype) for x in (prob.Q, prob.K, prob.V, prob.dO)), prob.scale,
                             prob.causal, keep_of=keep_of, rp=rp)
    res = pu.judge(f"dropout p={p_drop} {pu.describe(prob)}", {k: pu.to_f64(v) for k, v in got.items()}, exp, ref,
                   standard=False, dtype=prob.dtype, d=prob.d)
    return {k: v[0] for k, v in res.items()}


@pytest.mark.parametrize("causal", [False, True])
@pytest.mark.parametrize("p_drop", [0.1, 0.5])
@pytest.mark.parametrize("Nq,Nk,Hq,Hkv,d", [(1, 1, 2, 2, 64), (65, 65, 2, 2, 64), (128, 128, 2, 2, 128), (257, 300, 4, 2, 128),
                                            (300, 515, 2, 1, 64), (33, 1000, 8, 2, 128)])
def test_dropout_matches_the_oracle(Nq, Nk, Hq, Hkv, d, p_drop, causal):
    prob = inputs.make_cross(B=2, Nq=Nq, Nk=Nk, Hq=Hq, Hkv=Hkv, d=d, causal=causal, seed=6000 + Nq + Nk)
    check_dropout(prob, p_drop, seed=0x1234ABCD5678 + Nq)


@pytest.mark.parametrize("causal", [False, True])
@pytest.mark.parametrize("Nq,Nk,Hq,Hkv,d", [(65, 65, 2, 2, 64), (257, 300, 4, 2, 128), (300, 515, 2, 1, 64), (700, 700, 2, 2, 128)])
def test_dropout_in_half_precision(Nq, Nk, Hq, Hkv, d, causal):
    prob = inputs.make_cross(B=2, Nq=Nq, Nk=Nk, Hq=Hq, Hkv=Hkv, d=d, causal=causal, seed=6050 + Nq + Nk, dtype="f16")
    check_dropout(prob, 0.25, seed=0x77AA11 + Nk)


def test_zero_probability_reproduces_the_plain_entry_points_bitwise():
    prob = inputs.make_cross(B=2, Nq=200, Nk=260, Hq=4, Hkv=2, d=128, causal=True, seed=6100)
    got = run(prob, 0.0, 42)
    ref = pu.run_hip(prob)
    for nm in got:
        assert torch.equal(got[nm], ref[nm]), nm


def test_lse_does_not_depend_on_the_mask_and_the_mask_depends_on_the_seed():
    prob = inputs.make_cross(B=1, Nq=129, Nk=129, Hq=2, Hkv=2, d=64, causal=False, seed=6200)
    a, b, plain = run(prob, 0.25, 1), run(prob, 0.25, 2), pu.run_hip(prob)
    assert torch.equal(a["LSE"], plain["LSE"]) and torch.equal(b["LSE"], plain["LSE"])
    assert not torch.equal(a["O"], b["O"])
    again = run(prob, 0.25, 1)
    for nm in a:
        assert torch.equal(a[nm], again[nm]), nm  # same seed, same bits


def test_kept_fraction_seen_through_the_output():
    """V = all ones: every output element is (number of kept keys) / ((1 - p) Nk) for uniform P."""
    B, N, H, d = 1, 512, 2, 64
    Q = torch.zeros(B, N, H, d, dtype=torch.bfloat16, device="cuda")  # uniform probabilities
    K = torch.zeros_like(Q)
    V = torch.ones_like(Q)
    O, _ = binding.fa_dropout_fwd(Q, K, V, 0.125, False, 0.25, 7)
    torch.cuda.synchronize()
    thr = orc.dropout_threshold(0.25)
    for h in range(H):
        keep = orc.dropout_keep(7, h, N, N, thr)
        want = keep.sum(axis=1) / (0.75 * N)
        assert np.max(np.abs(pu.to_f64(O[0, :, h, 0]) - want)) <= 2 * pu.bf16_ulp(float(want.max()))


@pytest.mark.parametrize("Nq,Nk,d,causal", [(31, 255, 64, False), (64, 256, 128, True), (257, 257, 64, True),
                                            (33, 511, 128, False), (513, 513, 128, True), (1, 769, 64, False)])
def test_lengths_around_the_blocks_of_the_backward_on_small_grids(Nq, Nk, d, causal):
    """The dK/dV kernel's 128-key blocks that small grids take under dropout: a last block of 1, 127 or 128 keys, row
    tiles with a single row, wavefronts whose keys lie past the end or above every row."""
    check_dropout(inputs.make_cross(B=1, Nq=Nq, Nk=Nk, Hq=4, Hkv=2, d=d, causal=causal, seed=6300 + Nk), 0.1, seed=0x256)


def check_dropout_units(prob, p_drop, seed, units):
    """check_dropout on whole (sequence b, key/value head g) units of a larger dense batch."""
    Q, K, V, dO = (pu.to_gpu(x, prob.dtype) for x in (prob.Q, prob.K, prob.V, prob.dO))
    got = run(prob, p_drop, seed)
    widen = orc.widen_f16 if prob.dtype == "f16" else orc.widen_bf16
    thr = orc.dropout_threshold(p_drop)
    G = prob.Hq // prob.Hkv
    for t in got.values():
        assert torch.isfinite(t.float()).all()
    for (b, g) in units:
        k, v = widen(prob.K[b, :, g]), widen(prob.V[b, :, g])
        exp = {"O": [], "LSE": [], "dQ": [], "dK": np.zeros_like(k), "dV": np.zeros_like(v)}
        ref = {"O": [], "LSE": [], "dQ": [], "dK": np.zeros_like(k), "dV": np.zeros_like(v)}
        hs = slice(g * G, (g + 1) * G)
        for h in range(g * G, (g + 1) * G):
            keep = orc.dropout_keep(seed, b * prob.Hq + h, prob.N, prob.keys, thr)
            q, do = widen(prob.Q[b, :, h]), widen(prob.dO[b, :, h])
            o, lse, _ = orc.head_forward_dropout(q, k, v, prob.scale, prob.causal, keep, thr)
            dq, dk, dv = orc.head_backward_dropout(q, k, v, do, prob.scale, prob.causal, keep, thr)
            r = pu.reference_head(Q[b, :, h], K[b, :, g], V[b, :, g], dO[b, :, h], prob.scale, prob.causal,
                                  keep=torch.from_numpy(keep).cuda(), rp=256.0 / (256.0 - thr))
            for nm, x in (("O", o), ("LSE", lse), ("dQ", dq), ("dK", dk), ("dV", dv)):
                for to, value in ((exp, x), (ref, r[nm])):
                    if nm in ("dK", "dV"):
                        to[nm] += value
                    else:
                        to[nm].append(value)
        for nm in ("O", "LSE", "dQ"):
            exp[nm], ref[nm] = np.stack(exp[nm]), np.stack(ref[nm])
        part = {"O": pu.to_f64(got["O"][b, :, hs]).transpose(1, 0, 2), "LSE": pu.to_f64(got["LSE"][b, hs]),
                "dQ": pu.to_f64(got["dQ"][b, :, hs]).transpose(1, 0, 2), "dK": pu.to_f64(got["dK"][b, :, g]),
                "dV": pu.to_f64(got["dV"][b, :, g])}
        pu.judge(f"dropout p={p_drop} unit (b={b}, g={g}) {pu.describe(prob)}", part, exp, ref, standard=False, dtype=prob.dtype,
                 d=prob.d)


# (136 key/value heads over all sequences, 8 where the sequences are long: more than 256 workgroups, so the blocks are of
# 256 keys; at d = 64 with the mask that takes more than 4096 keys as well)
@pytest.mark.parametrize("dtype", ["bf16", "f16"])
@pytest.mark.parametrize("B,Nq,Nk,Hq,Hkv,d,causal", [
    (17, 100, 257, 8, 8, 64, False), (17, 33, 511, 16, 8, 64, False), (17, 1, 512, 8, 8, 64, False),
    (17, 100, 257, 8, 8, 128, False), (17, 33, 511, 16, 8, 128, False), (17, 1, 512, 8, 8, 128, False),
    (17, 257, 257, 8, 8, 128, True), (17, 100, 511, 16, 8, 128, True), (17, 512, 512, 8, 8, 128, True),
    (1, 4097, 4097, 8, 8, 64, True), (1, 100, 4351, 16, 8, 64, True), (2, 65, 4352, 4, 4, 64, True)])
def test_lengths_around_the_256_key_blocks_of_the_backward(B, Nq, Nk, Hq, Hkv, d, causal, dtype):
    """The dK/dV kernel's 256-key blocks under dropout: a last block of 1, 255 or 256 keys, row tiles with
    a single row, wavefronts whose keys lie past the end or above every row."""
    prob = inputs.make_cross(B=B, Nq=Nq, Nk=Nk, Hq=Hq, Hkv=Hkv, d=d, causal=causal, seed=6800 + Nk, dtype=dtype)
    check_dropout_units(prob, 0.1, 0x256, [(0, 0), (B - 1, Hkv - 1)])


@pytest.mark.parametrize("p_drop", [0.9, 255 / 256])
@pytest.mark.parametrize("Nq,Nk,d", [(200, 512, 64), (200, 512, 128), (512, 512, 64)])
def test_half_precision_gradients_at_a_high_probability(Nq, Nk, d, p_drop):
    """An output gradient of 2^-12: the entries of dS are subnormal half-precision numbers, spaced by 2^-24, as those of the
    reference are; rounded without their factor 1 / (1 - p) they would be spaced by that much more (a float64 model of
    the rounding: dQ off by 3.0e-7 and 2.1e-6 at p = 0.9, by 5e-7 and 5e-5 at 255/256)."""
    prob = inputs.make_cross(B=1, Nq=Nq, Nk=Nk, Hq=2, Hkv=2, d=d, causal=False, seed=6700 + Nq + d, dtype="f16")
    prob.dO = inputs.f32_to_f16_bits(orc.widen_f16(prob.dO).astype(np.float32) / 4096)
    check_dropout(prob, p_drop, seed=0xBEEF)


# (36 sequences x 8 heads fill more than 256 workgroups of 128 or 256 keys, one sequence does not; under the causal rule
# d = 64 takes the small form up to 4096 keys either way)
@pytest.mark.parametrize("causal", [False, True])
@pytest.mark.parametrize("N,Hq,Hkv,d", [(127, 8, 8, 64), (129, 8, 8, 64), (256, 8, 4, 64), (385, 8, 8, 64), (129, 8, 8, 128),
                                        (300, 16, 8, 128)])
def test_small_and_large_workgroups_of_the_backward_drop_the_same_entries(N, Hq, Hkv, d, causal):
    """The form of the dK/dV kernel is chosen by the size of the grid; the first sequence's results (its hash does not
    depend on the batch) are the same in a batch and alone, and alone they match the oracle. At d = 128 the small
    form adds dK and dV in two halves: float32 sums that differ by their own rounding end in the same 16-bit value
    or its neighbour (2^-7 of the value apart at most; values near zero are held to the sums' rounding instead)."""
    prob = inputs.make_dense(B=36, N=N, Hq=Hq, Hkv=Hkv, d=d, causal=causal, seed=6400 + N)
    Q, K, V, dO = (pu.to_gpu(x, prob.dtype) for x in (prob.Q, prob.K, prob.V, prob.dO))
    O, L = binding.fa_dropout_fwd(Q, K, V, prob.scale, causal, 0.2, 77)
    grads = binding.fa_dropout_bwd(Q, K, V, O, dO, L, prob.scale, causal, 0.2, 77)
    alone = binding.fa_dropout_bwd(*(x[:1].contiguous() for x in (Q, K, V, O, dO, L)), prob.scale, causal, 0.2, 77)
    for name, x, y in zip(("dQ", "dK", "dV"), grads, alone):
        if d == 64 or name == "dQ":
            assert torch.equal(x[0], y[0]), name
        else:
            torch.testing.assert_close(x[0].float(), y[0].float(), rtol=2.0 ** -7, atol=1e-4)
    check_dropout(inputs.make_dense(B=1, N=N, Hq=Hq, Hkv=Hkv, d=d, causal=causal, seed=6500 + N), 0.2, seed=77)


@pytest.mark.parametrize("causal", [False, True])
@pytest.mark.parametrize("dtype", ["bf16", "f16"])
@pytest.mark.parametrize("d,Hq,Hkv", [(64, 2, 2), (128, 4, 2)])
def test_ragged_batches_with_dropout(d, Hq, Hkv, causal, dtype):
    """fa_varlen_dropout_fwd / bwd against the oracle's ragged dropout: the generator counts rows and
    columns from the start of each sequence and uses sequence * Hq + head as its head index."""
    check_ragged_dropout(inputs.make_varlen([100, 257, 1, 31, 300], Hq=Hq, Hkv=Hkv, d=d, causal=causal, seed=6100 + d, dtype=dtype))


@pytest.mark.parametrize("causal", [False, True])
@pytest.mark.parametrize("dtype", ["bf16", "f16"])
@pytest.mark.parametrize("d", [64, 128])
def test_ragged_batches_with_dropout_on_large_grids(d, causal, dtype):
    """The same on grids of more than 256 workgroups by the longest sequence (forms.py has batches whose blocks themselves are as many)."""
    check_ragged_dropout(pu.large_varlen(d=d, causal=causal, seed=6900 + d, dtype=dtype))


def check_ragged_dropout(prob):
    causal, dtype, Hq, Hkv, d = prob.causal, prob.dtype, prob.Hq, prob.Hkv, prob.d
    Q, K, V, dO = (pu.to_gpu(x, dtype) for x in (prob.Q, prob.K, prob.V, prob.dO))
    cu, longest = torch.from_numpy(prob.cu_seqlens.astype(np.int32)).cuda(), int(prob.seqlens.max())
    p_drop, seed = 0.25, 0x1234567890ABCDEF
    O, L = binding.fa_varlen_dropout_fwd(Q, K, V, cu, longest, prob.scale, causal, p_drop, seed)
    dQ, dK, dV = binding.fa_varlen_dropout_bwd(Q, K, V, O, dO, L, cu, longest, prob.scale, causal, p_drop, seed)
    torch.cuda.synchronize()
    widen = orc.widen_f16 if dtype == "f16" else orc.widen_bf16
    Qf, Kf, Vf, dOf = (widen(x) for x in (prob.Q, prob.K, prob.V, prob.dO))
    eO, eL = orc.varlen_forward_dropout(Qf, Kf, Vf, prob.cu_seqlens, prob.scale, causal, p_drop, seed)
    edQ, edK, edV = orc.varlen_backward_dropout(Qf, Kf, Vf, dOf, prob.cu_seqlens, prob.scale, causal, p_drop, seed)
    keep_of, rp = keep_masks(seed, p_drop, Hq)
    ref = pu.reference_batch(Q, K, V, dO, prob.scale, causal, cu_q=prob.cu_seqlens, keep_of=keep_of, rp=rp)
    pu.judge(f"ragged dropout d{d} H{Hq}/{Hkv} causal={causal}",
             {nm: pu.to_f64(t) for nm, t in (("O", O), ("LSE", L), ("dQ", dQ), ("dK", dK), ("dV", dV))},
             dict(O=eO, LSE=eL, dQ=edQ, dK=edK, dV=edV), ref, standard=False, dtype=dtype, d=d)


@pytest.mark.timeout(600)
@pytest.mark.parametrize("name", ["dropout_d128_n8k_causal", "dropout_gqa_ragged"])
def test_full_size_dropout_workloads_sampled_units(name):
    """The benchmark shapes with dropout (p = 0.1): whole (sequence, head) units against the oracle
    and the 16-bit reference with the same keep mask; the ragged one on its shortest and longest
    sequence (grouped heads: dK, dV of a key/value head over its four query heads)."""
    prob = inputs.make_config(name)
    p_drop, seed = prob.meta["dropout"]
    thr = orc.dropout_threshold(p_drop)
    rp = 256.0 / (256.0 - thr)
    Q, K, V, dO = (pu.to_gpu(x) for x in (prob.Q, prob.K, prob.V, prob.dO))
    G = prob.Hq // prob.Hkv
    if prob.varlen:
        cu = torch.from_numpy(prob.cu_seqlens.astype(np.int32)).cuda()
        mx = int(prob.seqlens.max())
        O, L = binding.fa_varlen_dropout_fwd(Q, K, V, cu, mx, prob.scale, True, p_drop, seed)
        dQ, dK, dV = binding.fa_varlen_dropout_bwd(Q, K, V, O, dO, L, cu, mx, prob.scale, True, p_drop, seed)
        units = [(s, s % prob.Hkv, int(prob.cu_seqlens[s]), int(prob.cu_seqlens[s + 1]))
                 for s in sorted({int(np.argmin(prob.seqlens)), int(np.argmax(prob.seqlens))})]
    else:
        O, L = binding.fa_dropout_fwd(Q, K, V, prob.scale, True, p_drop, seed)
        dQ, dK, dV = binding.fa_dropout_bwd(Q, K, V, O, dO, L, prob.scale, True, p_drop, seed)
        units = [(0, 0, 0, prob.N), (prob.B - 1, prob.Hkv - 1, 0, prob.N)]
    torch.cuda.synchronize()
    for t in (O, L, dQ, dK, dV):
        assert torch.isfinite(t.float()).all()
    for (s, g, a, e) in units:
        n = e - a
        sel = (slice(a, e),) if prob.varlen else (s,)
        k, v = orc.widen_bf16(prob.K[sel][:, g]), orc.widen_bf16(prob.V[sel][:, g])
        exp = {"O": [], "LSE": [], "dQ": [], "dK": np.zeros_like(k), "dV": np.zeros_like(v)}
        ref = {"O": [], "LSE": [], "dQ": [], "dK": np.zeros_like(k), "dV": np.zeros_like(v)}
        for h in range(g * G, (g + 1) * G):
            keep = orc.dropout_keep(seed, s * prob.Hq + h, n, n, thr)
            q, do = orc.widen_bf16(prob.Q[sel][:, h]), orc.widen_bf16(prob.dO[sel][:, h])
            o, lse, _ = orc.head_forward_dropout(q, k, v, prob.scale, True, keep, thr)
            dq, dk, dv = orc.head_backward_dropout(q, k, v, do, prob.scale, True, keep, thr)
            r = pu.reference_head(Q[sel][:, h], K[sel][:, g], V[sel][:, g], dO[sel][:, h], prob.scale, True,
                                  keep=torch.from_numpy(keep).cuda(), rp=rp)
            for nm, x in (("O", o), ("LSE", lse), ("dQ", dq)):
                exp[nm].append(x)
                ref[nm].append(r[nm])
            exp["dK"] += dk
            exp["dV"] += dv
            ref["dK"] += r["dK"]
            ref["dV"] += r["dV"]
        hs = slice(g * G, (g + 1) * G)
        got = {"O": pu.to_f64(O[sel][:, hs]).transpose(1, 0, 2), "LSE": pu.to_f64(L[hs, a:e] if prob.varlen else L[s, hs]),
               "dQ": pu.to_f64(dQ[sel][:, hs]).transpose(1, 0, 2), "dK": pu.to_f64(dK[sel][:, g]), "dV": pu.to_f64(dV[sel][:, g])}
        for nm in ("O", "LSE", "dQ"):
            exp[nm], ref[nm] = np.stack(exp[nm]), np.stack(ref[nm])
        pu.judge(f"{name} unit (s={s}, g={g}, n={n})", got, exp, ref, standard=False, d=prob.d)
