"""Every instantiation of the backward kernels (forms.py) on the GPU: a sequence's gradients are those of the sequence alone, which takes
one of the small forms that the other tests hold against the oracle."""
import pytest

torch = pytest.importorskip("torch")

import forms
from paper_2307_08691_amd import binding

pytestmark = pytest.mark.gpu


def passes(kind, packed, causal, M, pattern, scale):
    """(forward, backward) of Q, K, V and, for packed batches, the offsets and the longest length."""
    extra = {"plain": (causal,), "window": forms.WINDOW, "dropout": (causal, forms.P_DROP, forms.SEED)}.get(kind)
    if kind == "mask":
        return (lambda q, k, v: binding.fa_mask_fwd(q, k, v, M, scale, causal),
                lambda q, k, v, o, g, l: binding.fa_mask_bwd(q, k, v, M, o, g, l, scale, causal))
    if kind == "blocks":
        return (lambda q, k, v: binding.fa_blocksparse_fwd(q, k, v, pattern, 64, scale, causal),
                lambda q, k, v, o, g, l: binding.fa_blocksparse_bwd(q, k, v, pattern, 64, o, g, l, scale, causal))
    fwd, bwd = {("plain", False): (binding.fa_cross_fwd, binding.fa_cross_bwd), ("plain", True): (binding.fa_varlen_fwd, binding.fa_varlen_bwd),
                ("window", False): (binding.fa_local_fwd, binding.fa_local_bwd),
                ("window", True): (binding.fa_varlen_local_fwd, binding.fa_varlen_local_bwd),
                ("dropout", False): (binding.fa_dropout_fwd, binding.fa_dropout_bwd),
                ("dropout", True): (binding.fa_varlen_dropout_fwd, binding.fa_varlen_dropout_bwd)}[kind, packed]
    return (lambda q, k, v, *at: fwd(q, k, v, *at, scale, *extra), lambda q, k, v, o, g, l, *at: bwd(q, k, v, o, g, l, *at, scale, *extra))


@pytest.mark.parametrize("dtype", ["bf16", "f16"])
@pytest.mark.parametrize("kind,packed,d,causal,B,N,Hq,Hkv", forms.cases())
def test_a_sequence_has_its_own_gradients_in_every_form(kind, packed, d, causal, B, N, Hq, Hkv, dtype):
    et, G = (torch.bfloat16 if dtype == "bf16" else torch.float16), Hq // Hkv
    g = torch.Generator(device="cuda").manual_seed(9900 + N + d + B)
    lens = forms.lengths(B, N) if packed else [N] * B
    cu = [0]
    for n in lens:
        cu.append(cu[-1] + n)
    Q, K, V, dO = (torch.randn((cu[-1], h, d), generator=g, device="cuda", dtype=et) for h in (Hq, Hkv, Hkv, Hq))
    M = pattern = None
    if kind == "mask":
        M = binding.mask_buffer(1, 1, N, N, "cuda", et)
        M.copy_(torch.randn(M.shape, generator=g, device="cuda", dtype=et))
    if kind == "blocks":
        nb = -(-N // 64)
        pattern = (torch.rand((1, 1, nb, nb), generator=g, device="cuda") < 0.6).to(torch.uint8)
    fwd, bwd = passes(kind, packed, causal, M, pattern, d ** -0.5)

    def run(q, k, v, do, nseq, at):
        if not packed:
            q, k, v, do = (x.view(nseq, N, -1, d) for x in (q, k, v, do))
        O, L = fwd(q, k, v, *at)
        return [x.reshape(-1, x.shape[-2], d) for x in bwd(q, k, v, O, do, L, *at)]

    offsets = lambda o: (torch.tensor(o, dtype=torch.int32, device="cuda"), max(b - a for a, b in zip(o, o[1:]))) if packed else ()
    whole = run(Q, K, V, dO, B, offsets(cu))
    assert all(torch.isfinite(x).all() for x in whole)
    # (the generator of dropout counts sequences and heads)
    units = [(0, 0)] if kind == "dropout" else [(0, 0), (B // 2, Hkv // 2), (B - 1, Hkv - 1)]
    for s, h in units:
        rows, qh, kh = slice(cu[s], cu[s + 1]), slice(h * G, (h + 1) * G), slice(h, h + 1)
        alone = run(*(x[rows, y].contiguous() for x, y in ((Q, qh), (K, kh), (V, kh), (dO, qh))), 1, offsets([0, lens[s]]))
        for name, x, y, heads in zip(("dQ", "dK", "dV"), whole, alone, (qh, kh, kh)):
            x = x[rows, heads]
            if kind == "dropout" and d == 128 and name != "dQ":
                # sums of a key's rows in two halves or in one chain: the same 16-bit value or its neighbour, values near zero apart by the
                # rounding of the sums (2^-24 of some hundred terms of order one)
                torch.testing.assert_close(x.float(), y.float(), rtol=2.0 ** (-7 if dtype == "bf16" else -10), atol=1e-3)
            else:
                assert torch.equal(x, y), (name, s, h)
