"""The work that users of this library have it do, as cases that can be timed.

Every case is one pass through the tensor-level entry points of paper_2307_08691_amd.binding, called
as the README shows: the caller holds the inputs, the entry point makes outputs and scratch. A training
case is a forward and a backward pass and returns O, the logsumexp and the three gradients; a serving
case is one forward call.

`path` says which entry points a case takes:
  dense     fa_fwd + fa_bwd (bfloat16) or fa_cross_fwd + fa_cross_bwd (half precision), one length
  ragged    fa_varlen_fwd + fa_varlen_bwd on a packed batch of uneven sequences
  dropout   fa_dropout_fwd + fa_dropout_bwd
  window    fa_local_fwd + fa_local_bwd
  prefill   fa_fwd alone: a prompt enters the model
  chunk     fa_kvcache_fwd, hundreds of new queries per sequence against a paged cache
  decode    fa_kvcache_fwd, one new query per sequence against a cache, paged or contiguous
  fp8       fa_fp8_fwd on E4M3 operands
"""
import math
import random

import torch

from paper_2307_08691_amd import binding


def listed():
    return [
        # The smallest training step that the tests run (one short sequence, two heads): launches and host time.
        dict(name="train_tiny", path="dense", dtype="bf16", B=1, N=128, Hq=2, Hkv=2, d=64, causal=False),
        # Many short sequences of the benchmark grid (16k tokens, hidden size 2048, N = 512, 32 heads of 64).
        dict(name="train_short", path="dense", dtype="bf16", B=32, N=512, Hq=32, Hkv=32, d=64, causal=True),
        # The headline training shape of the benchmark: two sequences of 8192 tokens, 16 heads of 128.
        dict(name="train_8k", path="dense", dtype="bf16", B=2, N=8192, Hq=16, Hkv=16, d=128, causal=True),
        # The grouped-query ragged training batch of the benchmark: 16 sequences of 256 .. 4096 tokens, packed.
        dict(name="train_ragged", path="ragged", dtype="bf16", nseq=16, lo=256, hi=4096, lens_seed=1005, Hq=32,
             Hkv=8, d=128, causal=True),
        # Encoder-style training in half precision: no causal rule, dropout on P, a length off every tile edge.
        dict(name="train_dropout", path="dropout", dtype="f16", B=4, N=1777, Hq=16, Hkv=16, d=64, causal=False,
             p_drop=0.1),
        # Sliding-window training: each token sees the newest 1024 of 8192.
        dict(name="train_window", path="window", dtype="bf16", B=2, N=8192, Hq=16, Hkv=16, d=128, left=1023, right=0),
        # Wide heads: 16k tokens in sequences of 2048, 8 heads of 256.
        dict(name="train_d256", path="dense", dtype="bf16", B=8, N=2048, Hq=8, Hkv=8, d=256, causal=True),
        # One prompt of an odd length enters a grouped-query model.
        dict(name="prefill_one", path="prefill", dtype="bf16", B=1, N=1531, Hq=32, Hkv=8, d=128, causal=True),
        # Chunked prefill in a serving engine: 512 new tokens for each of 4 sequences whose paged caches hold
        # up to 8192 tokens.
        dict(name="chunk_prefill", path="chunk", dtype="bf16", B=4, Nq=512, cap=8192, page=256, lens_seed=1006,
             Hq=32, Hkv=8, d=128, causal=True),
        # Decoding for a few users with short contexts: latency.
        dict(name="decode_small", path="decode", dtype="bf16", B=4, Nq=1, cap=2048, page=0, lens_seed=1008, Hq=32,
             Hkv=8, d=128, causal=True),
        # Decoding for a full serving batch: 64 sequences with up to 8192 cached tokens, paged: memory bandwidth.
        dict(name="decode_batch", path="decode", dtype="bf16", B=64, Nq=1, cap=8192, page=256, lens_seed=18600,
             Hq=32, Hkv=8, d=128, causal=True),
        # Prompt processing on FP8 operands, the benchmark shape.
        dict(name="prefill_fp8", path="fp8", B=2, N=8192, Hq=16, Hkv=16, d=128, causal=True),
    ]


# ---------------------------------------------------------------------------------------------
# more cases of the same ranges

def _log_int(rng, lo, hi):
    """An integer in lo .. hi, uniform over the logarithm; odd ones as likely as even ones."""
    return max(lo, min(hi, round(math.exp(rng.uniform(math.log(lo), math.log(hi))))))


def _length(rng, lo, hi):
    """A length: half of them rounded to a multiple of 64 as padded batches have them, half as they come."""
    n = _log_int(rng, lo, hi)
    return max(64, n // 64 * 64) if n >= 128 and rng.random() < 0.5 else n


def _heads(rng, most=32):
    hkv = rng.choice([h for h in (1, 2, 4, 8, 16, 32) if h <= most])
    return hkv * rng.choice([g for g in (1, 2, 4, 8) if hkv * g <= most]), hkv


def _draw_once(rng):
    path = rng.choice(["dense", "dense", "dense", "ragged", "dropout", "window", "prefill", "prefill", "chunk", "decode",
                       "decode", "fp8"])
    hq, hkv = _heads(rng)
    c = dict(path=path, dtype="bf16", Hq=hq, Hkv=hkv, d=rng.choice([64, 128]), causal=rng.random() < 0.7)
    if path == "dense":
        c.update(B=_log_int(rng, 1, 32), N=_length(rng, 64, 8192), d=rng.choice([64, 64, 96, 128, 128, 256]),
                 dtype=rng.choice(["bf16", "bf16", "f16"]))
    elif path == "ragged":
        hi = _log_int(rng, 256, 4096)
        c.update(nseq=_log_int(rng, 2, 32), lo=max(1, hi // 16), hi=hi, lens_seed=rng.randrange(1 << 30))
    elif path == "dropout":
        c.update(B=_log_int(rng, 1, 16), N=_length(rng, 128, 4096), p_drop=rng.choice([0.05, 0.1, 0.2]),
                 dtype=rng.choice(["bf16", "f16"]))
    elif path == "window":
        n = _length(rng, 1024, 8192)
        w = _log_int(rng, 64, n // 2)
        c.update(B=_log_int(rng, 1, 4), N=n, left=w - 1, right=rng.choice([0, 0, w - 1]))
        del c["causal"]
    elif path == "prefill":
        c.update(B=_log_int(rng, 1, 4), N=_length(rng, 64, 8192), causal=True)
    elif path == "chunk":
        cap = 256 * _log_int(rng, 8, 64)
        c.update(B=_log_int(rng, 1, 8), Nq=_log_int(rng, 64, 1024), cap=cap, page=rng.choice([64, 128, 256]),
                 lens_seed=rng.randrange(1 << 30), causal=True)
    elif path == "decode":
        c.update(B=_log_int(rng, 1, 96), Nq=1, cap=256 * _log_int(rng, 2, 64), page=rng.choice([0, 64, 256]),
                 lens_seed=rng.randrange(1 << 30), causal=True)
    else:  # fp8
        del c["dtype"]
        c.update(B=_log_int(rng, 1, 4), N=_length(rng, 256, 8192))
    return c


def draw(rng):
    limit = [max(w[k] for w in map(work, listed())) for k in ("bytes", "flops")]
    while True:
        c = _draw_once(rng)
        w = work(c)
        # (half of the largest listed work: narrow heads and dropout run below the largest case's rate)
        if w["bytes"] <= limit[0] and w["flops"] <= limit[1] / 2:
            return c


# ---------------------------------------------------------------------------------------------
# shapes

def _lengths(case):
    """Sequence lengths (ragged) or numbers of cached keys, the new ones among them (chunk, decode)."""
    r = random.Random(case["lens_seed"])
    if case["path"] == "ragged":
        return [r.randint(case["lo"], case["hi"]) for _ in range(case["nseq"])]
    lo = min(case["cap"], max(case["Nq"], case["cap"] // 64))
    lens = [r.randint(lo, case["cap"]) for _ in range(case["B"])]
    lens[0] = case["cap"]  # the longest sequence is what the cache was sized for
    return lens


def _pairs(nq, nk, causal):
    """Visible (query, key) pairs of one head; query r stands at position r + nk - nq."""
    return nq * nk - nq * (nq - 1) // 2 if causal else nq * nk


def _window_pairs(n, left, right):
    return sum(min(n - 1, q + right) - max(0, q - left) + 1 for q in range(n))


def work(case):
    path, d, hq, hkv = case["path"], case["d"], case["Hq"], case["Hkv"]
    if path == "ragged":
        lens = _lengths(case)
        tq = tk = sum(lens)
        pairs = sum(_pairs(n, n, case["causal"]) for n in lens)
    elif path in ("chunk", "decode"):
        lens = _lengths(case)
        tq, tk = case["B"] * case["Nq"], sum(lens)
        pairs = sum(_pairs(case["Nq"], n, case["causal"]) for n in lens)
    else:
        n, b = case["N"], case["B"]
        tq = tk = b * n
        pairs = b * (_window_pairs(n, case["left"], case["right"]) if path == "window" else _pairs(n, n, case["causal"]))
    fwd = 4.0 * d * hq * pairs
    stats = 4.0 * tq * hq  # the logsumexp, float32
    if path == "fp8":  # one byte per element in, two out
        return {"bytes": tq * hq * d * 3.0 + 2.0 * tk * hkv * d + stats, "flops": fwd}
    q, kv = 2.0 * tq * hq * d, 2.0 * tk * hkv * d
    if path in ("prefill", "chunk", "decode"):
        return {"bytes": 2 * q + 2 * kv + stats, "flops": fwd}
    # forward and backward: Q, K, V, dO in; O, logsumexp, dQ, dK, dV out; five products more
    return {"bytes": 4 * q + 4 * kv + stats, "flops": 3.5 * fwd}


# ---------------------------------------------------------------------------------------------
# inputs and passes

class _State:
    pass


def prepare(case, seed):
    g = torch.Generator(device="cuda").manual_seed(seed)
    path, d, hq, hkv = case["path"], case["d"], case["Hq"], case["Hkv"]
    dtype = torch.float16 if case.get("dtype") == "f16" else torch.bfloat16

    def normal(*shape):
        return torch.randn(shape, generator=g, device="cuda", dtype=dtype)

    s = _State()
    s.case, s.scale = case, d ** -0.5
    if path == "fp8":  # the usual amax scaling to E4M3, one scale per tensor
        eight, s.descale = [], []
        for h in (hq, hkv, hkv):
            x = torch.randn((case["B"], case["N"], h, d), generator=g, device="cuda")
            ds = float(x.abs().max()) / 448.0
            eight.append((x / ds).to(torch.float8_e4m3fn).view(torch.uint8))
            s.descale.append(ds)
        s.Q, s.K, s.V = eight[0], eight[1], binding.fp8_key_major(eight[2])
        return s
    if path == "ragged":
        lens = _lengths(case)
        cu = [0]
        for n in lens:
            cu.append(cu[-1] + n)
        s.cu, s.longest = torch.tensor(cu, dtype=torch.int32, device="cuda"), max(lens)
        s.Q, s.K, s.V, s.dO = (normal(cu[-1], h, d) for h in (hq, hkv, hkv, hq))
        return s
    if path in ("chunk", "decode"):
        b, cap, page = case["B"], case["cap"], case["page"]
        s.lens, s.table = torch.tensor(_lengths(case), dtype=torch.int32, device="cuda"), None
        s.Q = normal(b, case["Nq"], hq, d)
        if page:
            per_seq = cap // page
            s.K, s.V = normal(b * per_seq, page, hkv, d), normal(b * per_seq, page, hkv, d)
            s.table = torch.randperm(b * per_seq, generator=g, device="cuda").to(torch.int32).view(b, per_seq)
        else:
            s.K, s.V = normal(b, cap, hkv, d), normal(b, cap, hkv, d)
        return s
    b, n = case["B"], case["N"]
    s.Q, s.K, s.V = (normal(b, n, h, d) for h in (hq, hkv, hkv))
    if path != "prefill":
        s.dO = normal(b, n, hq, d)
    s.drop_seed = seed * 0x9E3779B1 % (1 << 63)
    return s


def run(s):
    c, path = s.case, s.case["path"]
    if path == "dense":
        fwd, bwd = ((binding.fa_cross_fwd, binding.fa_cross_bwd) if c["dtype"] == "f16" else
                    (binding.fa_fwd, binding.fa_bwd))
        O, L = fwd(s.Q, s.K, s.V, s.scale, c["causal"])
        return (O, L) + bwd(s.Q, s.K, s.V, O, s.dO, L, s.scale, c["causal"])
    if path == "ragged":
        O, L = binding.fa_varlen_fwd(s.Q, s.K, s.V, s.cu, s.longest, s.scale, c["causal"])
        return (O, L) + binding.fa_varlen_bwd(s.Q, s.K, s.V, O, s.dO, L, s.cu, s.longest, s.scale, c["causal"])
    if path == "dropout":
        O, L = binding.fa_dropout_fwd(s.Q, s.K, s.V, s.scale, c["causal"], c["p_drop"], s.drop_seed)
        return (O, L) + binding.fa_dropout_bwd(s.Q, s.K, s.V, O, s.dO, L, s.scale, c["causal"], c["p_drop"], s.drop_seed)
    if path == "window":
        O, L = binding.fa_local_fwd(s.Q, s.K, s.V, s.scale, c["left"], c["right"])
        return (O, L) + binding.fa_local_bwd(s.Q, s.K, s.V, O, s.dO, L, s.scale, c["left"], c["right"])
    if path == "prefill":
        return binding.fa_fwd(s.Q, s.K, s.V, s.scale, c["causal"])
    if path == "fp8":
        return binding.fa_fp8_fwd(s.Q, s.K, s.V, c["N"], s.scale, *s.descale, c["causal"])
    return binding.fa_kvcache_fwd(s.Q, s.K, s.V, s.scale, c["causal"], seqlens_k=s.lens, block_table=s.table)


def tolerance(case):
    # Measured against the same pass in float64 (2-norm of the error over 2-norm of the result, the largest
    # of O, dQ, dK, dV over the listed cases), stated about four times as large: bfloat16 2.7e-3 (its
    # rounding of the results and of P, dS as operands; half precision has three more bits), E4M3 2.2e-2
    # (the rounding of P). The logsumexp is off by 1e-7.
    if case["path"] == "fp8":
        return {"rel": 8e-2}
    return {"rel": 2e-3 if case["dtype"] == "f16" else 1e-2}
