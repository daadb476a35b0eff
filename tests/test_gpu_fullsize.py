"""GPU parity at the full benchmark sizes, in the launch configuration bench.py
times. The float64 oracle cannot materialise every (sequence, head) unit of
these workloads in seconds, so whole units are sampled (first and last head,
first and last sequence; shortest and longest sequence of the ragged batch) and
compared element by element; everything else is checked through properties that
hold at any size (finiteness, dV column sums)."""
import numpy as np
import pytest

from paper_2307_08691_amd import inputs
from oracle import attention_oracle as orc

pytestmark = pytest.mark.gpu

torch = pytest.importorskip("torch")
import parity_util as pu  # noqa: E402


check_units = pu.check_units


def global_properties(prob, got):
    for nm, t in got.items():
        assert torch.isfinite(t.float()).all(), f"{prob.name}: {nm} not finite"
    if not prob.varlen and prob.Hq == prob.Hkv:
        # rows of P sum to one => per (batch, head) the columns of dV sum to those of dO
        dO = pu.to_gpu(prob.dO).double().sum(dim=1)
        dV = got["dV"].double().sum(dim=1)
        scale = float(pu.to_gpu(prob.dO).double().abs().sum(dim=1).max())
        assert float((dO - dV).abs().max()) <= 4e-3 * scale


@pytest.mark.parametrize("name", ["d128_n8k_causal", "sweep_d64_n8192_full", "sweep_d64_n2048_causal",
                                  "sweep_d128_n512_full", "d96_n8k_causal", "d32_n8k_causal", "d256_n8k_causal"])
def test_dense_workloads_sampled_units(name):
    prob = inputs.make_config(name)
    got = pu.run_hip(prob)
    global_properties(prob, got)
    units = [(0, 0), (prob.B - 1, prob.Hkv - 1)]
    print(name, check_units(prob, got, units))


@pytest.mark.parametrize("dtype", ["bf16", "f16"])
@pytest.mark.parametrize("B,Nq,Nk,Hq,Hkv", [(1, 4097, 4097, 8, 8), (1, 8192, 8192, 8, 8), (2, 300, 4351, 8, 4), (1, 4352, 4352, 16, 8)])
def test_causal_batches_past_4096_keys_at_head_dimension_64(B, Nq, Nk, Hq, Hkv, dtype):
    """At d = 64 the causal dK/dV kernel has workgroups of four wavefronts up to 4096 keys and on grids that fit the
    compute units at once; longer sequences on larger grids, as these (264 workgroups of 128 keys or more), take
    those of eight: last blocks of 1, 255 and 256 keys. (Not seed 15600 + Nk: at Nk = 4352 row 2 of head 0, a row of
    three keys, has an O whose rounding to bfloat16 moves D = dO . O by 0.046 and with it dQ by 0.0174 = scale |dD|
    max|P K| in exact arithmetic; Algorithm 2 takes D from O, and the reference rounds another O.)"""
    prob = inputs.make_cross(B=B, Nq=Nq, Nk=Nk, Hq=Hq, Hkv=Hkv, d=64, causal=True, seed=15700 + Nk, dtype=dtype)
    got = pu.run_hip(prob)
    for nm, t in got.items():
        assert torch.isfinite(t.float()).all(), nm
    print(prob.name, check_units(prob, got, [(0, 0), (B - 1, Hkv - 1)]))


@pytest.mark.parametrize("dtype", ["bf16", "f16"])
@pytest.mark.parametrize("causal", [False, True])
@pytest.mark.parametrize("B,Nq,Nk,Hq,Hkv", [(4, 512, 512, 64, 64), (2, 1000, 1000, 64, 16), (8, 512, 512, 64, 8),
                                            (16, 300, 300, 64, 64), (2, 1024, 1024, 64, 64), (4, 512, 777, 64, 16)])
def test_short_sequences_in_chained_workgroups(B, Nq, Nk, Hq, Hkv, causal, dtype):
    """Dense d = 128 batches of short sequences whose forward pass runs in workgroups that take
    2, 4 or 8 (row block, head, sequence) items in a row, fetching an item's Q_i and first tiles
    while the previous one finishes: units from both ends and the middle of the batch, which sit
    at different places of different chains; ragged last row blocks (N = 1000, 300); more keys
    than queries."""
    prob = inputs.make_cross(B=B, Nq=Nq, Nk=Nk, Hq=Hq, Hkv=Hkv, d=128, causal=causal, seed=15000 + Nq + Hkv, dtype=dtype)
    got = pu.run_hip(prob)
    for nm, t in got.items():
        assert torch.isfinite(t.float()).all(), nm
    units = [(0, 0), (B // 2, Hkv // 2), (B - 1, Hkv - 1), (B - 1, 0), (0, Hkv - 1)]
    print(prob.name, check_units(prob, got, units))


def test_long_context_wide_range_sampled_units():
    prob = inputs.make_config("long_n16k_causal_x3")
    got = pu.run_hip(prob)
    global_properties(prob, got)
    print(prob.name, check_units(prob, got, [(0, 15)]))
    # sampled rows of another head, forward only (cheap: one row block of scores at a time)
    rows = np.asarray([0, 1, 127, 128, 8191, 8192, 16000, 16383])
    k = orc.widen_bf16(prob.K[0, :, 3])
    v = orc.widen_bf16(prob.V[0, :, 3])
    q = orc.widen_bf16(prob.Q[0, rows, 3])
    o, lse = orc.rows_forward(q, rows, k, v, prob.scale, True)
    Qg, Kg, Vg, dOg = (pu.to_gpu(x) for x in (prob.Q, prob.K, prob.V, prob.dO))
    ref = pu.reference_head(Qg[0, rows, 3], Kg[0, :, 3], Vg[0, :, 3], dOg[0, rows, 3], prob.scale, True, backward=False,
                            pos=rows)
    pu.judge(f"{prob.name} sampled rows of head 3", {"O": pu.to_f64(got["O"][0, rows, 3]), "LSE": pu.to_f64(got["LSE"][0, 3, rows])},
             {"O": o, "LSE": lse}, ref, standard=False, d=prob.d)


def test_gqa_ragged_sampled_sequences():
    prob = inputs.make_config("gqa_ragged")
    got = pu.run_hip(prob)
    for nm, t in got.items():
        assert torch.isfinite(t.float()).all(), nm
    lens = prob.seqlens
    cu = prob.cu_seqlens
    picks = sorted({int(np.argmin(lens)), int(np.argmax(lens)), 0, len(lens) - 1})
    G = prob.Hq // prob.Hkv
    Qg, Kg, Vg, dOg = (pu.to_gpu(x) for x in (prob.Q, prob.K, prob.V, prob.dO))
    for s in picks:
        a, e = int(cu[s]), int(cu[s + 1])
        g = s % prob.Hkv
        hs = slice(g * G, (g + 1) * G)
        Q = orc.widen_bf16(prob.Q[a:e, hs])[None]
        dO = orc.widen_bf16(prob.dO[a:e, hs])[None]
        K = orc.widen_bf16(prob.K[a:e, g:g + 1])[None]
        V = orc.widen_bf16(prob.V[a:e, g:g + 1])[None]
        exp = {}
        exp["O"], exp["LSE"] = orc.attention_forward(Q, K, V, prob.scale, True)
        exp["dQ"], exp["dK"], exp["dV"] = orc.attention_backward(Q, K, V, dO, prob.scale, True)
        ref = pu.reference_batch(Qg[a:e, hs][None], Kg[a:e, g:g + 1][None], Vg[a:e, g:g + 1][None], dOg[a:e, hs][None],
                                 prob.scale, True)
        gotu = {"O": got["O"][a:e, hs][None], "LSE": got["LSE"][hs, a:e][None], "dQ": got["dQ"][a:e, hs][None],
                "dK": got["dK"][a:e, g:g + 1][None], "dV": got["dV"][a:e, g:g + 1][None]}
        pu.judge(f"{prob.name} sequence {s} (len {e - a}) kv head {g}", {k: pu.to_f64(v) for k, v in gotu.items()}, exp, ref,
                 standard=True, d=prob.d)


@pytest.mark.timeout(900)
def test_tensors_beyond_two_to_the_31_elements():
    """Maximum sizes: 4 x 32768 x 128 heads x 128 = 2^31 elements (4 GiB) per tensor, so element
    offsets of the last sequences and heads do not fit 32 bits. Inputs are drawn on the GPU from a
    seeded generator (the host copy of a tensor this size would dominate the test); the last
    (sequence, head) unit is checked against the oracle on sampled query rows (O, L, dQ) and
    sampled key columns (dK, dV), whose row statistics the oracle computes blockwise for the whole
    head; the first unit on sampled rows."""
    from paper_2307_08691_amd import binding
    B, N, H, d, scale = 4, 32768, 128, 128, 128 ** -0.5
    gen = torch.Generator(device="cuda").manual_seed(7001)
    draw = lambda: torch.randn(B, N, H, d, device="cuda", dtype=torch.float32, generator=gen).to(torch.bfloat16)  # noqa: E731
    Q = draw()
    K = draw()
    V = draw()
    dO = draw()
    assert Q.numel() == 2 ** 31
    O, L = binding.fa_fwd(Q, K, V, scale, True)
    dQ, dK, dV = binding.fa_bwd(Q, K, V, O, dO, L, scale, True)
    torch.cuda.synchronize()
    rows = np.asarray([0, 1, 255, 256, 12345, 32766, 32767])
    cols = [0, 127, 128, 20000, 32767]
    f64 = lambda t: t.double().cpu().numpy()  # noqa: E731
    for (b, h, full) in ((B - 1, H - 1, True), (0, 0, False)):
        q, k, v, do = f64(Q[b, :, h]), f64(K[b, :, h]), f64(V[b, :, h]), f64(dO[b, :, h])
        exp, gotu = {}, {"O": f64(O[b, rows, h]), "LSE": f64(L[b, h, rows]), "dQ": f64(dQ[b, rows, h])}
        exp["O"], exp["LSE"] = orc.rows_forward(q[rows], rows, k, v, scale, True)
        exp["dQ"] = orc.rows_backward_dq(q[rows], rows, k, v, do[rows], scale, True)
        ref = pu.reference_head(Q[b, rows, h], K[b, :, h], V[b, :, h], dO[b, rows, h], scale, True, pos=rows)
        ref = {nm: ref[nm] for nm in gotu}
        if full:
            Lall, _, Dall = orc.head_statistics_blockwise(q, k, v, do, scale, True, block=1024)
            exp["dK"], exp["dV"] = orc.cols_backward_dkdv(q, k[cols], v[cols], cols, N, do, Lall, Dall, scale, True)
            whole = pu.reference_head(Q[b, :, h], K[b, :, h], V[b, :, h], dO[b, :, h], scale, True)
            ref.update(dK=whole["dK"][cols], dV=whole["dV"][cols])
            gotu.update(dK=f64(dK[b, cols, h]), dV=f64(dV[b, cols, h]))
            del whole
        pu.judge(f"2^31 elements, unit ({b},{h}), sampled rows and columns", gotu, exp, ref, standard=True, d=d)
    for t in (O, L, dQ, dK, dV):
        # finiteness of everything, in slices (a 4 GiB tensor widened at once would double the footprint)
        for b in range(B):
            assert torch.isfinite(t[b].float()).all()


@pytest.mark.parametrize("name", ["d128_n8k_causal", "sweep_d64_n8192_full", "sweep_d128_n512_causal"])
def test_repeated_full_size_calls_give_the_same_bits(name):
    """No atomics and no order that depends on timing: five forward + backward passes over a full-size
    workload (all compute units busy, workgroups finishing in varying order) produce identical bits.
    A missing wait or barrier in the kernels' hand-ordered LDS traffic would show here as a difference."""
    prob = inputs.make_config(name)
    first = pu.run_hip(prob)
    for _ in range(4):
        again = pu.run_hip(prob)
        for nm in first:
            assert torch.equal(first[nm], again[nm]), nm
