"""The native marshalling of the usual calls (csrc/fa_host.cpp): it makes the call that binding.py would make, and leaves
whatever is not an ordinary call to it."""
import itertools
import sys
import types

import pytest

from paper_2307_08691_amd import binding

torch = pytest.importorskip("torch")


@pytest.fixture(scope="module")
def host():
    binding._load_host()
    assert binding._host, "the extension module has not been built"
    return binding._host


def test_shares_of_a_cache_are_those_of_the_binding(host):
    for B, (Hq, Hkv), Nq, Nk, d, ragged in itertools.product(
            (1, 2, 5, 64, 128, 129, 500), ((1, 1), (8, 2), (32, 8), (32, 1)), (1, 2, 32, 33, 70, 512, 1000),
            (1, 64, 768, 960, 1023, 1024, 1216, 2304, 5000, 8192, 8300, 70000), (64, 96, 128), (False, True)):
        want = binding._cache_splits(B, Hq, Hkv, Nq, Nk, d, ragged)
        assert host.cache_splits(B, Hq, Hkv, Nq, Nk, d, ragged) == want, (B, Hq, Hkv, Nq, Nk, d, ragged)


def test_host_tensors_and_other_objects_are_left_to_the_binding(host):
    x = torch.zeros(1, 64, 2, 64, dtype=torch.bfloat16)
    assert host.dense_fwd(0, x, x, x, 0.125, True) is None
    assert host.dense_fwd(0, None, 1, "x", 0.125, True) is None
    assert host.dense_fwd() is None and host.dense_bwd() is None and host.varlen_fwd() is None
    assert host.varlen_bwd() is None and host.kvcache_fwd() is None
    with pytest.raises(ValueError):
        binding.fa_fwd(x, x, x, 0.125, True)


def test_an_extension_that_does_not_load_is_reported_and_left_alone(host, monkeypatch):
    monkeypatch.setitem(sys.modules, binding.__package__ + "._host", None)  # its import raises ImportError
    monkeypatch.setattr(binding, "_host", None)
    with pytest.warns(RuntimeWarning, match="does not load"):
        binding._load_host()
    assert binding._host is False  # looked for once; the calls are made in Python


def test_a_build_without_the_extension_still_makes_the_library(monkeypatch, tmp_path, capsys):
    from paper_2307_08691_amd import build as fa_build
    stale = tmp_path / "_host.so"
    stale.write_bytes(b"of an earlier build")

    def no_compiler():
        raise RuntimeError("no C++ compiler")

    linked = []
    monkeypatch.setattr(fa_build, "HOST_LIB", str(stale))
    monkeypatch.setattr(fa_build, "build_host", no_compiler)
    monkeypatch.setattr(fa_build, "_compile", lambda source, obj: "")
    monkeypatch.setattr(fa_build.subprocess, "run", lambda cmd, **kw: linked.append(cmd) or types.SimpleNamespace(returncode=0, stderr=""))
    assert fa_build.build() == fa_build.LIB and len(linked) == 1
    assert not stale.exists() and "no C++ compiler" in capsys.readouterr().err


def test_after_a_build_nothing_of_the_old_library_is_called(host, monkeypatch):
    import __graft_entry__
    from paper_2307_08691_amd import build as fa_build
    monkeypatch.setattr(fa_build, "build", lambda verbose=False: fa_build.LIB)
    old = binding.load()
    __graft_entry__.build()
    assert binding._host is None and binding.load() is not old


def _calls(dtype):
    """name -> (native call, the same through the Python of the binding: outputs passed in)."""
    g = torch.Generator(device="cuda").manual_seed(22000)
    t = lambda *s: torch.randn(s, generator=g, device="cuda", dtype=dtype)
    e = torch.empty_like
    Q, K, V, dO = t(2, 200, 4, 64), t(2, 200, 2, 64), t(2, 200, 2, 64), t(2, 200, 4, 64)
    P = [x.view(400, -1, 64) for x in (Q, K, V)]
    cu = torch.tensor([0, 130, 400], dtype=torch.int32, device="cuda")
    L, Lp = (torch.empty(s, device="cuda") for s in ((2, 4, 200), (4, 400)))
    out = {}

    def both(name, fwd, bwd, ops, stat, args):
        f = lambda: fwd(*ops, *args)
        out[name] = (f, lambda: fwd(*ops, *args, O=e(ops[0]), LSE=e(stat)))
        O, l = f()
        g_ = dO.view_as(O)
        head = (ops + [O, g_, l]) if isinstance(ops, list) else list(ops) + [O, g_, l]
        out[name + " backward"] = (lambda: bwd(*head, *args), lambda: bwd(*head, *args, dQ=e(ops[0])))

    if dtype == torch.bfloat16:
        both("plain", binding.fa_fwd, binding.fa_bwd, [Q, K, V], L, (0.125, True))
    both("cross", binding.fa_cross_fwd, binding.fa_cross_bwd, [Q, K[:, :150].contiguous(), V[:, :150].contiguous()], L, (0.125, False))
    both("dropout", binding.fa_dropout_fwd, binding.fa_dropout_bwd, [Q, K, V], L, (0.125, True, 0.1, (1 << 63) + 5))
    both("window", binding.fa_local_fwd, binding.fa_local_bwd, [Q, K, V], L, (0.125, 20, -1))
    both("packed", binding.fa_varlen_fwd, binding.fa_varlen_bwd, P, Lp, (cu, 270, 0.125, True))
    q, lens = Q[:, :1].contiguous(), torch.tensor([70, 200], dtype=torch.int32, device="cuda")
    pools = [x.repeat(1, 3, 1, 1)[:, :512].reshape(8, 128, 2, 64).contiguous() for x in (K, V)]
    table = torch.tensor([[3, 0, 6, 1], [2, 7, 5, 4]], dtype=torch.int32, device="cuda")
    for name, kv, kw in (("cache", [K, V], {}), ("cache with lengths", [K, V], dict(seqlens_k=lens)),
                         ("paged cache", pools, dict(seqlens_k=lens, block_table=table)),
                         ("paged cache, bounded", pools, dict(seqlens_k=lens, block_table=table, max_seqlen_k=200))):
        f = lambda kv=kv, kw=kw, **o: binding.fa_kvcache_fwd(q, *kv, 0.125, True, **kw, **o)
        out[name] = (f, lambda f=f: f(O=e(q)))
    return out


@pytest.mark.gpu
@pytest.mark.parametrize("dtype", [torch.bfloat16, torch.float16])
def test_native_and_python_calls_agree_bitwise(host, dtype, monkeypatch):
    class Counting:
        def __init__(self):
            self.native = 0

        def __getattr__(self, name):
            def call(*args):
                r = getattr(host, name)(*args)
                self.native += r is not None
                return r
            return call

    for name, (native, python) in _calls(dtype).items():
        count = Counting()
        monkeypatch.setattr(binding, "_host", count)
        got = native()
        assert count.native == 1, f"{name} did not go through the native path"
        want = python()
        assert count.native == 1
        assert len(got) == len(want)
        for x, y in zip(got, want):
            assert x.dtype == y.dtype and x.shape == y.shape and torch.equal(x.view(torch.uint8), y.view(torch.uint8)), name


@pytest.mark.gpu
def test_what_is_not_an_ordinary_call_keeps_its_answer(host):
    Q = torch.randn(2, 200, 4, 64, device="cuda", dtype=torch.bfloat16)
    K = torch.randn(2, 200, 2, 64, device="cuda", dtype=torch.bfloat16)
    O, L = binding.fa_fwd(Q, K, K, 0.125, True)
    for bad in (Q.transpose(1, 2), Q.half(), Q[:, :100].contiguous(), Q.cpu(), Q[..., :60].contiguous()):
        assert host.dense_fwd(0, bad, K, K, 0.125, True) is None
    for bad in (K[:1], K.half(), K.cpu(), K[..., :32].contiguous(), K[:, ::2]):
        assert host.dense_fwd(0, Q, K, bad, 0.125, True) is None
        with pytest.raises(ValueError):
            binding.fa_fwd(Q, K, bad, 0.125, True)
    assert host.dense_fwd(0, Q, K, K, 0.125, 1) is None and host.dense_fwd(0, Q, K, K, 1, True) is None  # (the binding takes them)
    assert torch.equal(binding.fa_fwd(Q, K, K, 0.125, 1)[0], O)
    assert host.dense_fwd(0, torch.nn.Parameter(Q), K, K, 0.125, True) is not None
    class Sub(torch.Tensor):
        pass
    assert host.dense_fwd(0, Q.as_subclass(Sub), K, K, 0.125, True) is None
    from torch.utils._python_dispatch import TorchDispatchMode
    class Mode(TorchDispatchMode):
        def __torch_dispatch__(self, func, types, args=(), kwargs=None):
            return func(*args, **(kwargs or {}))
    with Mode():
        assert host.dense_fwd(0, Q, K, K, 0.125, True) is None
        assert torch.equal(binding.fa_fwd(Q, K, K, 0.125, True)[0], O)
    seen = []
    torch.func.vmap(lambda s: seen.append(host.dense_fwd(0, Q, K, K, 0.125, True)) or s)(torch.zeros(2, device="cuda"))
    assert seen == [None]
    # another stream than the default one: the call goes where torch's current stream is
    st = torch.cuda.Stream()
    st.wait_stream(torch.cuda.current_stream())
    with torch.cuda.stream(st):
        o, l = binding.fa_fwd(Q, K, K, 0.125, True)
    torch.cuda.synchronize()
    assert torch.equal(o, O) and torch.equal(l, L)
