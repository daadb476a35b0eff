"""GPU parity: the HIP path, called through the C ABI binding, against the
float64 oracle on the same seeded bf16 inputs, element by element.

Bars (bf16 inputs ~ N(0,1)): max|dO| <= 2e-2, max|d(dQ,dK,dV)| <= 5e-2,
max|dLSE| <= 1e-3 against the oracle, and in every case the error must not
exceed that of a bf16 implementation that materialises S and P (section 2.2's
standard implementation) by more than one bf16 ulp at the tensor's largest
magnitude (parity_util.judge).
"""
import numpy as np
import pytest

from paper_2307_08691_amd import binding, inputs
from oracle import attention_oracle as orc

pytestmark = pytest.mark.gpu

torch = pytest.importorskip("torch")
import parity_util as pu  # noqa: E402


check = pu.check


def test_tiny_config_exact_shape():
    prob = inputs.make_config("tiny")
    errs = check(prob)
    print("tiny", errs)


@pytest.mark.parametrize("causal", [False, True])
@pytest.mark.parametrize("d", [64, 128])
@pytest.mark.parametrize("N", [1, 2, 31, 63, 64, 65, 127, 128, 129, 257, 300, 515])
def test_ragged_tail_lengths(N, d, causal):
    prob = inputs.make_dense(B=2, N=N, Hq=2, Hkv=2, d=d, causal=causal, seed=2000 + N)
    check(prob)


@pytest.mark.parametrize("causal", [False, True])
@pytest.mark.parametrize("d,Hq,Hkv", [(64, 4, 2), (128, 8, 2), (128, 4, 1), (64, 6, 6)])
def test_grouped_query_heads(d, Hq, Hkv, causal):
    prob = inputs.make_dense(B=2, N=200, Hq=Hq, Hkv=Hkv, d=d, causal=causal, seed=2100 + Hq)
    check(prob)


@pytest.mark.parametrize("causal", [False, True])
def test_several_row_and_column_blocks(causal):
    prob = inputs.make_dense(B=1, N=1100, Hq=3, Hkv=3, d=128, causal=causal, seed=2200)
    check(prob)
    prob = inputs.make_dense(B=1, N=900, Hq=2, Hkv=1, d=64, causal=causal, seed=2201)
    check(prob)


def test_wide_score_range():
    # Q, K scaled by 3 before rounding: scores ~ N(0, 9^2 / sqrt(d) scale), LSE in the tens
    prob = inputs.make_dense(B=1, N=700, Hq=2, Hkv=2, d=128, causal=True, seed=2300, qk_mult=3.0)
    errs = check(prob)
    print("wide", errs)


def test_nonstandard_scale():
    prob = inputs.make_dense(B=1, N=260, Hq=2, Hkv=2, d=64, causal=False, seed=2400, scale=0.05)
    check(prob)
    prob = inputs.make_dense(B=1, N=260, Hq=2, Hkv=2, d=64, causal=True, seed=2401, scale=0.3)
    check(prob)


@pytest.mark.parametrize("causal", [False, True])
@pytest.mark.parametrize("d,Hq,Hkv", [(128, 8, 2), (64, 4, 4)])
def test_packed_ragged_batch(d, Hq, Hkv, causal):
    lens = [5, 130, 0, 64, 257, 1, 300, 128]
    prob = inputs.make_varlen(lens, Hq=Hq, Hkv=Hkv, d=d, causal=causal, seed=2500)
    check(prob)


# (number of sequences, longest, Hq, Hkv, d): 16 and 130 query heads x sequences per XCD with gaps on every
# level, head counts that are no multiple of 8, one pair per XCD and fewer, more pairs than the kernels number
# without gaps (264 per XCD, for the row blocks only and for both), one length for all, an empty batch entry
@pytest.mark.parametrize("causal", [False, True])
@pytest.mark.parametrize("nseq,longest,Hq,Hkv,d", [(16, 900, 8, 2, 128), (65, 300, 16, 8, 64), (7, 1100, 6, 3, 64),
                                                   (3, 1025, 2, 1, 128), (33, 270, 64, 8, 64), (132, 260, 16, 16, 64),
                                                   (5, 400, 4, 2, 256), (9, 520, 4, 4, 96)])
def test_ragged_batches_are_covered_without_gaps(nseq, longest, Hq, Hkv, d, causal):
    """Every row of every sequence is computed exactly once whatever order the blocks are handed out in."""
    rng = np.random.default_rng(9100 + nseq)
    lens = rng.integers(0, longest + 1, nseq)
    lens[nseq // 2], lens[0] = longest, 0
    prob = inputs.make_varlen(lens, Hq=Hq, Hkv=Hkv, d=d, causal=causal, seed=9200 + nseq)
    Q, K, V, dO = (pu.to_gpu(x, prob.dtype) for x in (prob.Q, prob.K, prob.V, prob.dO))
    cu, mx = torch.from_numpy(prob.cu_seqlens.astype(np.int32)).cuda(), min(longest + 300, int(lens.sum()))
    bad = lambda x: torch.full_like(x, float("nan"))
    O, L = binding.fa_varlen_fwd(Q, K, V, cu, mx, prob.scale, causal, O=bad(Q),
                                 LSE=torch.full((Hq, Q.shape[0]), float("nan"), device="cuda"))
    grads = binding.fa_varlen_bwd(Q, K, V, O, dO, L, cu, mx, prob.scale, causal, dQ=bad(Q), dK=bad(K), dV=bad(V))
    for s in range(nseq):
        a, e = int(prob.cu_seqlens[s]), int(prob.cu_seqlens[s + 1])
        if a == e:
            continue
        q, k, v, g = (x[a:e].unsqueeze(0).contiguous() for x in (Q, K, V, dO))
        o, l = binding.fa_fwd(q, k, v, prob.scale, causal)
        want = (o, l) + binding.fa_bwd(q, k, v, o, g, l, prob.scale, causal)
        for name, x, y in zip(("O", "LSE", "dQ", "dK", "dV"), (O[a:e], L[:, a:e]) + tuple(t[a:e] for t in grads), want):
            assert torch.equal(x, y[0]), f"{name} of sequence {s} ({e - a} tokens)"


@pytest.mark.parametrize("causal", [False, True])
@pytest.mark.parametrize("dtype", ["bf16", "f16"])
@pytest.mark.parametrize("d", [64, 128])
def test_packed_ragged_batches_on_large_grids(d, dtype, causal):
    """More workgroups than compute units: both backward kernels in their forms of eight wavefronts."""
    check(pu.large_varlen(d=d, causal=causal, seed=9370 + d, dtype=dtype))


def test_packed_ragged_equals_dense_calls_bitwise():
    """A packed batch of equal lengths must reproduce the dense entry point bit for bit
    (every output is deterministic)."""
    prob = inputs.make_dense(B=3, N=200, Hq=4, Hkv=2, d=128, causal=True, seed=2600)
    dense = pu.run_hip(prob)
    packed = inputs.AttnProblem(name="packed", Q=prob.Q.reshape(600, 4, 128), K=prob.K.reshape(600, 2, 128),
                                V=prob.V.reshape(600, 2, 128), dO=prob.dO.reshape(600, 4, 128), Hq=4, Hkv=2, d=128,
                                scale=prob.scale, causal=True,
                                cu_seqlens=np.asarray([0, 200, 400, 600], dtype=np.int32))
    rag = pu.run_hip(packed)
    assert torch.equal(dense["O"].reshape(600, 4, 128), rag["O"])
    assert torch.equal(dense["LSE"].permute(1, 0, 2).reshape(4, 600), rag["LSE"])
    assert torch.equal(dense["dK"].reshape(600, 2, 128), rag["dK"])
    assert torch.equal(dense["dV"].reshape(600, 2, 128), rag["dV"])
    assert torch.equal(dense["dQ"].reshape(600, 4, 128), rag["dQ"])


# (lengths on either side of the 128- and 256-row blocks; 36 sequences x 8 heads fill more than 256 workgroups
# of either size, one sequence does not. Of the kernels of four wavefronts and eight, these compare the dQ kernel at d = 64
# except for 257 and 640 tokens, the dK/dV kernel without the mask except for 640; test_forms_of_the_backward_agree_bitwise
# has the rest)
@pytest.mark.parametrize("causal", [False, True])
@pytest.mark.parametrize("N,Hq,Hkv,d", [(128, 8, 8, 64), (129, 8, 8, 64), (256, 8, 8, 64), (257, 8, 4, 64), (385, 8, 8, 64),
                                        (640, 8, 8, 64), (129, 8, 8, 128), (300, 16, 8, 128)])
def test_small_and_large_workgroups_agree_bitwise(N, Hq, Hkv, d, causal):
    """The form of the backward kernels is chosen by the size of the grid; a sequence's results do not depend on it."""
    prob = inputs.make_dense(B=36, N=N, Hq=Hq, Hkv=Hkv, d=d, causal=causal, seed=9300 + N)
    Q, K, V, dO = (pu.to_gpu(x, prob.dtype) for x in (prob.Q, prob.K, prob.V, prob.dO))
    O, L = binding.fa_fwd(Q, K, V, prob.scale, causal)

    def two_kernels(q, k, v, o, do, lse):  # (fa_bwd may take one kernel for short sequences; this entry point does not)
        grads = [torch.empty_like(x) for x in (q, k, v)]
        ws = torch.empty(binding.fa_bwd_workspace_bytes(q.shape[0], Hq, Hkv, N, d), dtype=torch.uint8, device="cuda")
        binding.fa_bwd_stages(q, k, v, o, do, lse, prob.scale, causal, 7, *grads, ws)
        return grads

    if d == 64:
        assert (large_workgroups(N, 36 * Hq, False) != large_workgroups(N, Hq, False)) == (N not in (257, 640))
        assert causal or (large_workgroups(N, 36 * Hkv, False) != large_workgroups(N, Hkv, False)) == (N != 640)
    grads = two_kernels(Q, K, V, O, dO, L)
    for s in (0, 17, 35):
        alone = two_kernels(*(x[s:s + 1].contiguous() for x in (Q, K, V, O, dO, L)))
        for name, x, y in zip(("dQ", "dK", "dV"), grads, alone):
            assert torch.equal(x[s], y[0]), name


def four_wavefronts(N, Nk, pairs, d, causal):
    """Whether the plain forward pass takes its form of four wavefronts: N queries on Nk keys, (sequence, query head) pairs."""
    small = -(-N // 128) * pairs
    if N <= 128 or small <= 256:
        return True
    if causal and Nk <= (4 if d == 64 else 2) * N:
        return small <= (768 if d == 64 else 512)
    return not (causal and d == 128) and 512 < small <= 768 and Nk <= (8 if causal else 16) * N


def whole_and_single(N, Nk, B, Hq, Hkv, d, grow, dtype, causal, last_value=None):
    """B sequences, which take the forward form of eight wavefronts, and some of them alone, which take that of four:
    [(O, L of the sequence in the batch, O, L alone)]."""
    assert four_wavefronts(N, Nk, Hq, d, causal) and not four_wavefronts(N, Nk, B * Hq, d, causal)
    g = torch.Generator(device="cuda").manual_seed(9370 + N + Nk)
    et = torch.bfloat16 if dtype == "bf16" else torch.float16
    Q, K, V = (torch.randn(s, generator=g, device="cuda", dtype=et) for s in ((B, N, Hq, d), (B, Nk, Hkv, d), (B, Nk, Hkv, d)))
    K *= torch.linspace(1, grow, Nk, device="cuda").view(1, Nk, 1, 1).to(et)
    if last_value is not None:
        V[:, Nk - 1] = last_value
    O, L = binding.fa_cross_fwd(Q, K, V, d ** -0.5, causal)
    alone = lambda s: binding.fa_cross_fwd(*(x[s:s + 1].contiguous() for x in (Q, K, V)), d ** -0.5, causal)
    return [(O[s], L[s], *(x[0] for x in alone(s))) for s in (0, B // 2, B - 1)]


# (both sides of every edge of the four-wavefront forward kernel: blocks of 128 rows, 64 keys, wavefronts of 32 rows that see
# fewer blocks than their workgroup; `grow` = 8 so that the reference of the softmax moves in the middle of a row; two lengths,
# on either side of the ratios that the choice of the form goes by: with 2, 4, 8 and 16 times as many keys as queries, and more)
@pytest.mark.parametrize("causal", [False, True])
@pytest.mark.parametrize("dtype", ["bf16", "f16"])
@pytest.mark.parametrize("N,Nk,B,Hq,Hkv,d,grow", [(129, 129, 72, 8, 8, 64, 1), (192, 192, 72, 8, 4, 128, 1), (257, 257, 48, 8, 8, 128, 8),
                                                 (320, 320, 48, 8, 2, 64, 8), (449, 449, 40, 8, 8, 128, 1),
                                                 (130, 511, 72, 8, 8, 128, 1), (200, 263, 72, 8, 8, 64, 1),
                                                 (129, 259, 24, 8, 8, 128, 1), (160, 641, 24, 8, 4, 64, 8),
                                                 (129, 2065, 40, 8, 2, 64, 1)])
def test_forms_of_the_forward_pass_agree_bitwise(N, Nk, B, Hq, Hkv, d, grow, dtype, causal):
    """The form of the forward kernel is chosen by the size of the grid; a sequence's results do not depend on it."""
    for O, L, o, l in whole_and_single(N, Nk, B, Hq, Hkv, d, grow, dtype, causal):
        assert torch.isfinite(O).all() and torch.isfinite(L).all() and torch.equal(O, o) and torch.equal(L, l)


@pytest.mark.parametrize("dtype", ["bf16", "f16"])
@pytest.mark.parametrize("N,Nk,B,Hq,Hkv,d", [(257, 257, 48, 8, 8, 128), (320, 320, 48, 8, 2, 64)])
def test_forms_of_the_forward_pass_keep_an_infinite_value_to_the_same_rows(N, Nk, B, Hq, Hkv, d, dtype):
    """The last key's value is infinite: under the causal rule the rows that visit no block of 64 keys with it stay clear of
    it, and both forms agree on which rows those are."""
    for O, L, o, l in whole_and_single(N, Nk, B, Hq, Hkv, d, 1, dtype, True, float("inf")):
        assert torch.isfinite(O[:(Nk - 1) // 64 * 64]).all() and not torch.isfinite(O[-1]).any()
        assert torch.equal(O.view(torch.int16), o.view(torch.int16)) and torch.equal(L, l)


def large_workgroups(n, pairs, short_too):
    """Whether a backward kernel at d = 64 takes its form of eight wavefronts: n rows (keys), (sequence, head) pairs;
    short_too in the causal dK/dV kernel."""
    small, large = -(-n // 128) * pairs, -(-n // 256) * pairs
    return small > 256 and not (short_too and n <= 4096) and not (large >= 512 and 10 * large >= 6 * small)


# B sequences against their first `part`: the form differs in the dQ and in the dK/dV kernel as (dq, dkdv) says.
@pytest.mark.parametrize("B,part,N,Hq,Hkv,causal,dq,dkdv", [
    (36, 17, 257, 8, 8, False, True, True),   # four wavefronts where blocks of 256 rows would be mostly padding
    (36, 17, 640, 8, 8, False, True, True),
    (36, 17, 257, 8, 8, True, True, False),
    (17, 1, 640, 8, 8, False, True, True),    # ... and where the grid fits the compute units at once
    (17, 1, 1025, 8, 4, True, True, False),
    (2, 1, 4097, 4, 4, True, True, True),     # the causal dK/dV kernel of eight wavefronts: past 4096 keys
    (2, 1, 4352, 8, 4, True, False, True)])
@pytest.mark.parametrize("p_drop", [0.0, 0.2])
def test_forms_of_the_backward_agree_bitwise(B, part, N, Hq, Hkv, causal, dq, dkdv, p_drop):
    """At d = 64 a sequence's gradients do not depend on the form that the size of the batch chooses."""
    assert dq == (large_workgroups(N, B * Hq, False) != large_workgroups(N, part * Hq, False))
    assert dkdv == (large_workgroups(N, B * Hkv, causal) != large_workgroups(N, part * Hkv, causal))
    prob = inputs.make_dense(B=B, N=N, Hq=Hq, Hkv=Hkv, d=64, causal=causal, seed=9350 + N)
    Q, K, V, dO = (pu.to_gpu(x, prob.dtype) for x in (prob.Q, prob.K, prob.V, prob.dO))
    O, L = binding.fa_dropout_fwd(Q, K, V, prob.scale, causal, p_drop, 78)
    whole = binding.fa_dropout_bwd(Q, K, V, O, dO, L, prob.scale, causal, p_drop, 78)
    some = binding.fa_dropout_bwd(*(x[:part].contiguous() for x in (Q, K, V, O, dO, L)), prob.scale, causal, p_drop, 78)
    for name, x, y in zip(("dQ", "dK", "dV"), whole, some):
        assert torch.equal(x[:part], y), name


# (lengths on either side of the pieces of 32 keys, the row tiles of 64 and the three sizes of workgroup; 256 pairs or more take the
# one-kernel form, a few with shared heads, or beyond 256 tokens, the two kernels; without shared heads and up to 192 tokens
# every grid takes the former, which the oracle judges above)
@pytest.mark.parametrize("causal", [False, True])
@pytest.mark.parametrize("dtype", ["bf16", "f16"])
@pytest.mark.parametrize("packed", [False, True])
@pytest.mark.parametrize("N,B,Hq,Hkv", [(1, 32, 16, 8), (33, 32, 16, 8), (64, 64, 8, 4), (127, 64, 32, 4), (129, 32, 16, 8),
                                        (256, 64, 32, 4), (257, 32, 8, 8), (415, 32, 8, 8), (512, 32, 8, 8)])
def test_one_kernel_backward_agrees_bitwise(N, B, Hq, Hkv, packed, dtype, causal):
    """The backward of short sequences at d = 64 is one kernel or two by the size of the grid; a sequence's gradients do not
    depend on it."""
    g = torch.Generator(device="cuda").manual_seed(9390 + N)
    et = torch.bfloat16 if dtype == "bf16" else torch.float16
    lens = [N] * B
    if packed:  # uneven, empty ones among them, the longest as long as the bound
        lens = [N] + torch.randint(0, N + 1, (B - 1,), generator=torch.Generator().manual_seed(N)).tolist()
    cu = [0]
    for n in lens:
        cu.append(cu[-1] + n)
    Q, K, V, dO = (torch.randn((cu[-1], h, 64), generator=g, device="cuda", dtype=et) for h in (Hq, Hkv, Hkv, Hq))
    if packed:
        cut = torch.tensor(cu, dtype=torch.int32, device="cuda")
        O, L = binding.fa_varlen_fwd(Q, K, V, cut, N, 0.125, causal)
        grads = binding.fa_varlen_bwd(Q, K, V, O, dO, L, cut, N, 0.125, causal)
        L = L.transpose(0, 1)
    else:
        dense = lambda x: x.view(B, N, -1, 64)
        O, L = binding.fa_cross_fwd(*map(dense, (Q, K, V)), 0.125, causal)
        grads = [x.view(B * N, -1, 64) for x in binding.fa_cross_bwd(*map(dense, (Q, K, V, O, dO)), L, 0.125, causal)]
        O, L = O.view(B * N, Hq, 64), L.transpose(1, 2).reshape(B * N, Hq)
    assert all(torch.isfinite(x).all() for x in grads)
    for s in (0, 1, B // 2, B - 1):
        a, e = cu[s], cu[s + 1]
        if a == e:
            continue
        q, k, v, o, do = (x[a:e].unsqueeze(0).contiguous() for x in (Q, K, V, O, dO))
        alone = binding.fa_cross_bwd(q, k, v, o, do, L[a:e].transpose(0, 1).unsqueeze(0).contiguous(), 0.125, causal)
        for name, x, y in zip(("dQ", "dK", "dV"), grads, alone):
            assert torch.equal(x[a:e].view(torch.int16), y[0].view(torch.int16)), (name, s, e - a)


# (one pair, and three and ten: past the last full set of eight XCDs; as many blocks of 128 and of 256 rows as make an XCD that
# holds them all hold more than fit on it at once, and fewer)
@pytest.mark.parametrize("causal", [False, True])
@pytest.mark.parametrize("packed", [False, True])
@pytest.mark.parametrize("H,N,d", [(1, 8321, 64), (3, 8321, 64), (10, 4300, 64), (10, 300, 64), (1, 8300, 128), (3, 8300, 128),
                                   (10, 4300, 128), (3, 4300, 256)])
def test_pairs_that_do_not_divide_over_the_xcds(H, N, d, packed, causal):
    """The blocks of pairs past the last full set of eight are dealt to all XCDs: every block is computed, by whichever workgroup,
    and a head's results are those of the head alone."""
    g = torch.Generator(device="cuda").manual_seed(9500 + N + H)
    Q, K, V, dO = (torch.randn((N, H, d), generator=g, device="cuda", dtype=torch.bfloat16) for _ in range(4))
    cu = [0, N // 3, N // 3 + 5, N] if packed else [0, N]
    cut = torch.tensor(cu, dtype=torch.int32, device="cuda")
    longest = max(b - a for a, b in zip(cu, cu[1:]))

    def run(h0, h1):
        q, k, v, do = (x[:, h0:h1].contiguous() for x in (Q, K, V, dO))
        bad = lambda x: torch.full_like(x, float("nan"))
        lse = torch.full((h1 - h0, N), float("nan"), device="cuda")
        if packed:
            O, L = binding.fa_varlen_fwd(q, k, v, cut, longest, d ** -0.5, causal, O=bad(q), LSE=lse)
            grads = binding.fa_varlen_bwd(q, k, v, O, do, L, cut, longest, d ** -0.5, causal, dQ=bad(q), dK=bad(k), dV=bad(v))
            return (O, L.transpose(0, 1)) + tuple(grads)
        one = lambda x: x.view(1, *x.shape)
        O, L = binding.fa_fwd(one(q), one(k), one(v), d ** -0.5, causal, O=bad(one(q)), LSE=one(lse))
        grads = binding.fa_bwd(one(q), one(k), one(v), O, one(do), L, d ** -0.5, causal, dQ=bad(one(q)), dK=bad(one(k)), dV=bad(one(v)))
        return (O[0], L[0].transpose(0, 1)) + tuple(x[0] for x in grads)

    whole = run(0, H)
    assert all(torch.isfinite(x).all() for x in whole)
    for h in {0, H // 2, H - 1}:
        for name, x, y in zip(("O", "LSE", "dQ", "dK", "dV"), whole, run(h, h + 1)):
            assert torch.equal(x[:, h], y[:, 0]), (name, h)


# (512 pairs: blocks of 256 rows, or of 128 in the forms of four wavefronts and among the mask's keys, that fill rounds of the chip
# without a rest take two launches; one sequence of them takes one grid)
@pytest.mark.parametrize("kind,d,N,causal", [("plain", 128, 300, False), ("plain", 128, 512, True), ("plain", 96, 257, True),
                                             ("plain", 80, 400, False), ("plain", 104, 511, True), ("plain", 48, 300, False),
                                             ("plain", 32, 510, True), ("plain", 64, 300, False), ("plain", 64, 600, True),
                                             ("window", 128, 400, False), ("window", 64, 300, False), ("dropout", 64, 390, True),
                                             ("dropout", 64, 512, False), ("mask", 128, 300, True), ("mask", 64, 500, False),
                                             ("blocks", 128, 512, False), ("blocks", 64, 512, True)])
@pytest.mark.parametrize("dtype", ["bf16", "f16"])
def test_one_grid_and_two_launches_agree_bitwise(kind, d, N, causal, dtype):
    """The backward is a pre-pass and one grid, or two kernels, by how the blocks divide over the chip; a sequence's gradients do
    not depend on it."""
    B, H, scale = 64, 8, d ** -0.5
    g = torch.Generator(device="cuda").manual_seed(9700 + N + d)
    et = torch.bfloat16 if dtype == "bf16" else torch.float16
    Q, K, V, dO = (torch.randn((B, N, H, d), generator=g, device="cuda", dtype=et) for _ in range(4))
    M = binding.mask_buffer(1, 1, N, N, "cuda", et) if kind == "mask" else None
    if kind == "mask":
        M.copy_(torch.randn(M.shape, generator=g, device="cuda", dtype=et))
    nb = -(-N // 64)
    pattern = (torch.rand((1, H, nb, nb), generator=g, device="cuda") < 0.5).to(torch.uint8) if kind == "blocks" else None
    fwd, bwd = {
        "plain": (lambda q, k, v: binding.fa_cross_fwd(q, k, v, scale, causal),
                  lambda q, k, v, o, do, l: binding.fa_cross_bwd(q, k, v, o, do, l, scale, causal)),
        "window": (lambda q, k, v: binding.fa_local_fwd(q, k, v, scale, 100, 30),
                   lambda q, k, v, o, do, l: binding.fa_local_bwd(q, k, v, o, do, l, scale, 100, 30)),
        "dropout": (lambda q, k, v: binding.fa_dropout_fwd(q, k, v, scale, causal, 0.2, 78),
                    lambda q, k, v, o, do, l: binding.fa_dropout_bwd(q, k, v, o, do, l, scale, causal, 0.2, 78)),
        "mask": (lambda q, k, v: binding.fa_mask_fwd(q, k, v, M, scale, causal),
                 lambda q, k, v, o, do, l: binding.fa_mask_bwd(q, k, v, M, o, do, l, scale, causal)),
        "blocks": (lambda q, k, v: binding.fa_blocksparse_fwd(q, k, v, pattern, 64, scale, causal),
                   lambda q, k, v, o, do, l: binding.fa_blocksparse_bwd(q, k, v, pattern, 64, o, do, l, scale, causal)),
    }[kind]
    O, L = fwd(Q, K, V)
    whole = bwd(Q, K, V, O, dO, L)
    alone = bwd(*(x[:1].contiguous() for x in (Q, K, V, O, dO, L)))  # (the first: the generator of dropout counts sequences)
    for name, x, y in zip(("dQ", "dK", "dV"), whole, alone):
        assert torch.isfinite(x).all() and torch.equal(x[0], y[0]), name


# (eight heads to a key/value head, or four: a block of keys is a chain of hundreds of row tiles, which several workgroups share unless the
# workspace holds D alone; lengths off the tiles, fewer tiles than shares in a packed batch's short sequences, every product width)
@pytest.mark.parametrize("packed", [False, True])
@pytest.mark.parametrize("kind,d,N,Hkv,causal", [("plain", 128, 700, 1, False), ("plain", 128, 1301, 2, True), ("plain", 96, 511, 1, True),
                                                 ("plain", 96, 640, 1, False), ("plain", 120, 600, 1, True), ("plain", 104, 513, 1, False),
                                                 ("plain", 64, 1100, 1, True), ("plain", 64, 1250, 2, False), ("plain", 32, 900, 1, True),
                                                 ("plain", 24, 800, 1, False), ("plain", 48, 900, 1, True), ("plain", 40, 700, 1, False),
                                                 ("window", 128, 900, 1, False), ("window", 64, 1300, 1, False),
                                                 ("dropout", 128, 520, 1, True), ("dropout", 128, 700, 1, False),
                                                 ("dropout", 64, 1000, 1, True), ("dropout", 64, 800, 1, False)])
@pytest.mark.parametrize("dtype", ["bf16", "f16"])
def test_shares_of_a_block_of_keys(kind, d, N, Hkv, causal, dtype, packed):
    """dK and dV added from the shares' float32 sums are the single chain's, apart from the order of the sums: the same 16-bit
    value or its neighbour (2^-7 or 2^-10 of the value apart at most; values near zero are held to the sums' rounding, 2^-24 of some
    thousand terms below one). dQ, which has no shares, is the same."""
    G, scale = 8 // Hkv, d ** -0.5
    et = torch.bfloat16 if dtype == "bf16" else torch.float16
    g = torch.Generator(device="cuda").manual_seed(9800 + N + d)
    cu = [0, N, N, N + 5, N + 5 + N // 3] if packed else [0, N, 2 * N]
    T = cu[-1]
    Q, K, V, dO = (torch.randn((T, h, d), generator=g, device="cuda", dtype=et) for h in (G * Hkv, Hkv, Hkv, G * Hkv))
    cut = torch.tensor(cu, dtype=torch.int32, device="cuda")
    if packed:
        extra = {"plain": (causal,), "window": (300, 50), "dropout": (causal, 0.2, 78)}[kind]
        fwd, bwd = {"plain": (binding.fa_varlen_fwd, binding.fa_varlen_bwd), "window": (binding.fa_varlen_local_fwd, binding.fa_varlen_local_bwd),
                    "dropout": (binding.fa_varlen_dropout_fwd, binding.fa_varlen_dropout_bwd)}[kind]
        shape, lengths, need = (lambda x: x), (cut, N), binding.fa_varlen_bwd_workspace_bytes(T, G * Hkv, Hkv, d)
    else:
        extra = {"plain": (causal,), "window": (300, 50), "dropout": (causal, 0.2, 78)}[kind]
        fwd, bwd = {"plain": (binding.fa_cross_fwd, binding.fa_cross_bwd), "window": (binding.fa_local_fwd, binding.fa_local_bwd),
                    "dropout": (binding.fa_dropout_fwd, binding.fa_dropout_bwd)}[kind]
        shape, lengths, need = (lambda x: x.view(2, N, -1, d)), (), binding.fa_cross_bwd_workspace_bytes(2, G * Hkv, Hkv, N, N, d)
    Q, K, V, dO = map(shape, (Q, K, V, dO))
    O, L = fwd(Q, K, V, *lengths, scale, *extra)
    just_d = (4 * T * G * Hkv + 255) // 256 * 256
    assert need > just_d

    def grads(nbytes):
        ws = torch.full((nbytes + 256,), 255, dtype=torch.uint8, device="cuda")  # NaN as float32
        r = bwd(Q, K, V, O, dO, L, *lengths, scale, *extra, workspace=ws[:nbytes], **{n: torch.full_like(x, float("nan")) for n, x in
                                                                                     (("dQ", Q), ("dK", K), ("dV", V))})
        assert (ws[nbytes:] == 255).all()
        return r

    whole, shared = grads(just_d), grads(need)
    assert torch.equal(whole[0], shared[0]) and not torch.equal(whole[1], shared[1])
    for x, y in zip(whole[1:], shared[1:]):
        torch.testing.assert_close(y.float(), x.float(), rtol=2.0 ** (-7 if et == torch.bfloat16 else -10), atol=1e-3)


def test_shares_match_the_oracle_and_need_no_workspace():
    prob = inputs.make_dense(B=1, N=513, Hq=8, Hkv=1, d=128, causal=True, seed=9850)
    check(prob)
    Q, K, V, dO = (pu.to_gpu(x, prob.dtype) for x in (prob.Q, prob.K, prob.V, prob.dO))
    O, L = binding.fa_fwd(Q, K, V, prob.scale, True)
    want = binding.fa_bwd(Q, K, V, O, dO, L, prob.scale, True)
    got = [torch.full_like(x, float("nan")) for x in (Q, K, V)]
    binding.fa_bwd_noalloc(Q, K, V, O, dO, L, prob.scale, True, *got)
    for x, y in zip(want, got):
        assert torch.equal(x, y)


@pytest.mark.parametrize("d", [64, 128])
def test_cache_and_fp8_pairs_that_do_not_divide_over_the_xcds(d):
    """As above for the split-key kernel (nine pairs, more shares than an XCD holds) and the FP8 kernel."""
    g = torch.Generator(device="cuda").manual_seed(9600 + d)
    Q, K, V = (torch.randn(s, generator=g, device="cuda", dtype=torch.bfloat16)
               for s in ((3, 700, 3, d), (3, 1500, 3, d), (3, 1500, 3, d)))
    lens = torch.tensor([1500, 900, 1300], dtype=torch.int32, device="cuda")
    O, L = binding.fa_kvcache_fwd(Q, K, V, d ** -0.5, True, seqlens_k=lens, num_splits=12)
    for s in range(3):
        o, l = binding.fa_kvcache_fwd(*(x[s:s + 1] for x in (Q, K, V)), d ** -0.5, True, seqlens_k=lens[s:s + 1], num_splits=12)
        assert torch.isfinite(O[s]).all() and torch.equal(O[s], o[0]) and torch.equal(L[s], l[0])
    N = 8400 if d == 128 else 16700
    q, k, v = ((torch.randn((1, N, 2, d), generator=g, device="cuda") * 16).to(torch.float8_e4m3fn).view(torch.uint8) for _ in range(3))
    O, L = binding.fa_fp8_fwd(q, k, binding.fp8_key_major(v), N, d ** -0.5, 0.06, 0.06, 0.06, True)
    for h in range(2):
        one = [x[:, :, h:h + 1].contiguous() for x in (q, k, v)]
        o, l = binding.fa_fp8_fwd(one[0], one[1], binding.fp8_key_major(one[2]), N, d ** -0.5, 0.06, 0.06, 0.06, True)
        assert torch.isfinite(O).all() and torch.equal(O[:, :, h], o[:, :, 0]) and torch.equal(L[:, h], l[:, 0])


# (the grids on which each form of the two kernels is chosen: every small one, the small dK/dV form beside the large dQ
# form, both large ones; every product width of a padded head dimension and d = 256)
@pytest.mark.parametrize("order", [(1, 6), (1, 2, 4), (1, 4, 2), (3, 4), (5, 2)])
@pytest.mark.parametrize("B,N,Hq,Hkv,d,causal", [(1, 257, 4, 2, 64, True), (1, 257, 4, 2, 64, False), (1, 300, 4, 2, 128, True),
                                                 (1, 300, 4, 4, 128, False), (36, 256, 8, 8, 64, True),
                                                 (36, 256, 8, 8, 64, False), (40, 256, 8, 8, 128, True),
                                                 (1, 200, 2, 1, 96, True), (1, 200, 2, 1, 96, False), (1, 200, 2, 1, 32, True),
                                                 (1, 200, 2, 1, 32, False), (1, 200, 2, 1, 48, True), (1, 200, 2, 1, 48, False),
                                                 (1, 200, 2, 1, 104, True), (1, 200, 2, 1, 104, False), (1, 200, 2, 1, 256, True),
                                                 (1, 200, 2, 1, 256, False)])
def test_any_split_of_the_backward_into_stages(B, N, Hq, Hkv, d, causal, order):
    """fa_bwd_stages runs whatever subset of the three stages it is asked for: the pre-pass first and the two
    kernels together, apart or in either order write all of dQ, dK and dV, to the bit as fa_bwd does: D is the same chain of
    sums whether the pre-pass or the dQ kernel forms it."""
    prob = inputs.make_dense(B=B, N=N, Hq=Hq, Hkv=Hkv, d=d, causal=causal, seed=9400 + N + d)
    Q, K, V, dO = (pu.to_gpu(x, prob.dtype) for x in (prob.Q, prob.K, prob.V, prob.dO))
    O, L = binding.fa_fwd(Q, K, V, prob.scale, causal)
    want = binding.fa_bwd(Q, K, V, O, dO, L, prob.scale, causal)
    got = [torch.full_like(x, float("nan")) for x in (Q, K, V)]
    ws = torch.empty(binding.fa_bwd_workspace_bytes(B, Hq, Hkv, N, d), dtype=torch.uint8, device="cuda")
    for stages in order:
        binding.fa_bwd_stages(Q, K, V, O, dO, L, prob.scale, causal, stages, *got, ws)
    for name, x, y in zip(("dQ", "dK", "dV"), got, want):
        assert torch.isfinite(x).all(), f"{name} not written"
        assert torch.equal(x, y), name


# (shapes that fa_bwd hands to one kernel, to two of four and of eight wavefronts, d = 128, padded heads, d = 256)
@pytest.mark.parametrize("B,N,Hq,Hkv,d,causal", [(1, 100, 2, 2, 64, False), (64, 100, 8, 4, 64, True), (40, 200, 8, 8, 64, False),
                                                 (25, 450, 8, 8, 64, True), (1, 450, 4, 2, 64, True), (8, 1100, 8, 8, 64, False),
                                                 (2, 300, 4, 2, 128, True), (1, 200, 2, 1, 96, False), (1, 200, 2, 1, 256, True)])
def test_single_stages_after_a_whole_backward(B, N, Hq, Hkv, d, causal):
    """Asked for all three stages, fa_bwd_stages leaves D in the workspace as well: a later stage on the same arguments reads
    it there and repeats its part of the results, which are those of fa_bwd, bit for bit."""
    prob = inputs.make_dense(B=B, N=N, Hq=Hq, Hkv=Hkv, d=d, causal=causal, seed=9450 + N + d)
    Q, K, V, dO = (pu.to_gpu(x, prob.dtype) for x in (prob.Q, prob.K, prob.V, prob.dO))
    O, L = binding.fa_fwd(Q, K, V, prob.scale, causal)
    ws = torch.full((binding.fa_bwd_workspace_bytes(B, Hq, Hkv, N, d),), 255, dtype=torch.uint8, device="cuda")  # NaN as float32
    want = binding.fa_bwd(Q, K, V, O, dO, L, prob.scale, causal)
    whole = [torch.empty_like(x) for x in (Q, K, V)]
    binding.fa_bwd_stages(Q, K, V, O, dO, L, prob.scale, causal, 7, *whole, ws)
    got = [torch.full_like(x, float("nan")) for x in (Q, K, V)]
    for stages in (2, 4):
        binding.fa_bwd_stages(Q, K, V, O, dO, L, prob.scale, causal, stages, *got, ws)
    for name, x, y, z in zip(("dQ", "dK", "dV"), got, whole, want):
        assert torch.isfinite(z).all() and torch.equal(x, z) and torch.equal(y, z), name


@pytest.mark.parametrize("d", [64, 128])
def test_every_output_is_bit_reproducible(d):
    """No output is accumulated by atomic adds (dQ comes from a row-block pass of its own instead
    of section 3.2's atomic accumulation), so two runs on the same inputs agree bit for bit:
    the deterministic backward."""
    prob = inputs.make_dense(B=2, N=1333, Hq=4, Hkv=2, d=d, causal=True, seed=2700 + d)
    a = pu.run_hip(prob)
    b = pu.run_hip(prob)
    for nm in ("O", "LSE", "dQ", "dK", "dV"):
        assert torch.equal(a[nm], b[nm]), nm


def test_outputs_stay_inside_their_buffers():
    """Poisoned guard rows on both sides of every output must survive (tail blocks)."""
    from paper_2307_08691_amd import binding
    B, N, H, d, pad = 2, 130, 2, 64, 64
    prob = inputs.make_dense(B=B, N=N, Hq=H, Hkv=H, d=d, causal=True, seed=2800)
    Q, K, V, dO = (pu.to_gpu(x) for x in (prob.Q, prob.K, prob.V, prob.dO))

    def guarded(shape, dtype):
        n = int(np.prod(shape))
        buf = torch.full((n + 2 * pad * d,), float("nan"), dtype=dtype, device="cuda")
        return buf, buf[pad * d: pad * d + n].view(*shape)

    bO, O = guarded((B, N, H, d), torch.bfloat16)
    bL, L = guarded((B, H, N), torch.float32)
    binding.fa_fwd(Q, K, V, prob.scale, True, O=O, LSE=L)
    bufs = [bO, bL]
    outs = []
    for _ in range(3):
        bb, t = guarded((B, N, H, d), torch.bfloat16)
        bufs.append(bb)
        outs.append(t)
    binding.fa_bwd(Q, K, V, O, dO, L, prob.scale, True, dQ=outs[0], dK=outs[1], dV=outs[2])
    torch.cuda.synchronize()
    for bb in bufs:
        assert torch.isnan(bb[: pad * d]).all() and torch.isnan(bb[-pad * d:]).all()
    for t in [O, L] + outs:
        assert torch.isfinite(t.float()).all()


def test_closed_forms_on_the_gpu():
    """Q = 0 => O is the (prefix) mean of V and LSE = log(count); constant V => O = V."""
    prob = inputs.make_dense(B=1, N=200, Hq=2, Hkv=2, d=64, causal=True, seed=2900)
    prob.Q[...] = 0
    got = pu.run_hip(prob, backward=False)
    v = orc.widen_bf16(prob.V)[0]
    prefix = np.cumsum(v, axis=0) / np.arange(1, 201)[:, None, None]
    assert pu.maxdiff(pu.to_f64(got["O"])[0], prefix) <= 2e-2
    lse = pu.to_f64(got["LSE"])[0]
    assert pu.maxdiff(lse, np.tile(np.log(np.arange(1, 201)), (2, 1))) <= 1e-3
    prob2 = inputs.make_dense(B=1, N=200, Hq=2, Hkv=2, d=64, causal=False, seed=2901)
    prob2.V[...] = prob2.V[:, :1]
    got = pu.run_hip(prob2, backward=False)
    vv = orc.widen_bf16(prob2.V)
    assert pu.maxdiff(pu.to_f64(got["O"]), vv) <= pu.bf16_ulp(float(np.abs(vv).max()))


@pytest.mark.gpu
def test_mfma_probe_runs_and_reports_a_plausible_rate():
    """The register-resident MFMA loop: bounded by the datasheet rate at the clock it reports."""
    for rnd in (False, True):
        tf, ghz = binding.fa_mfma_probe(500, rnd)
        assert 0.5 < ghz < 2.6
        peak_at_clock = 256 * 4 * 1024 * ghz / 1e3  # TFLOP/s: 1024 FLOPs per SIMD and cycle
        assert 0.3 * peak_at_clock < tf < 1.05 * peak_at_clock


@pytest.mark.gpu
def test_forward_and_backward_replay_from_a_captured_graph():
    """The library allocates nothing and enqueues plain kernel launches on the caller's stream, so a
    whole step can be captured into a HIP graph. Replays (with other eager work and synchronisation
    in between, and new input values in the same buffers) must reproduce the eager results bit for bit."""
    import torch
    prob = inputs.make_dense(B=2, N=300, Hq=4, Hkv=2, d=128, causal=True, seed=2900)
    Q, K, V, dO = (pu.to_gpu(x) for x in (prob.Q, prob.K, prob.V, prob.dO))
    B, N, Hq, d = Q.shape
    O, L = torch.empty_like(Q), torch.empty(B, Hq, N, device="cuda")
    dQ, dK, dV = torch.empty_like(Q), torch.empty_like(K), torch.empty_like(V)
    ws = torch.empty(binding.fa_bwd_workspace_bytes(B, Hq, prob.Hkv, N, d), dtype=torch.uint8, device="cuda")

    def step():
        binding.fa_fwd(Q, K, V, prob.scale, True, O=O, LSE=L)
        binding.fa_bwd(Q, K, V, O, dO, L, prob.scale, True, dQ=dQ, dK=dK, dV=dV, workspace=ws)

    side = torch.cuda.Stream()
    side.wait_stream(torch.cuda.current_stream())
    with torch.cuda.stream(side):
        step()  # warm-up outside capture
    torch.cuda.current_stream().wait_stream(side)
    torch.cuda.synchronize()
    graph = torch.cuda.CUDAGraph()
    with torch.cuda.graph(graph):
        step()
    for trial in range(3):
        if trial:  # new values in the captured buffers
            Q.copy_(torch.randn_like(Q))
            dO.copy_(torch.randn_like(dO))
        step()
        torch.cuda.synchronize()
        eager = [t.clone() for t in (O, L, dQ, dK, dV)]
        for t in (O, L, dQ, dK, dV):
            t.fill_(float("nan"))
        graph.replay()
        torch.cuda.synchronize()
        for a, b in zip(eager, (O, L, dQ, dK, dV)):
            assert torch.equal(a, b)
