"""Problems by which every instantiation of the backward kernels is launched: each (kind, packed batch, head dimensions, causal,
[(sequences, longest length, query heads, key/value heads)]), in both element types. test_dispatch.py holds on the CPU that they reach
every kernel, test_gpu_forms.py runs them."""
from launches import P

FORMS = [
    ("blocks", False, (64, 128), False, [(40, 129, 4, 4), (2, 129, 1, 1)]),
    ("dropout", False, (64,), False, [(96, 129, 2, 2), (2, 129, 1, 1), (300, 129, 2, 2), (96, 257, 4, 4)]),
    ("dropout", False, (128,), False, [(3, 129, 32, 32), (2, 129, 1, 1), (40, 129, 4, 4), (40, 161, 4, 4)]),
    ("dropout", False, (64,), True, [(16, 129, 32, 32), (2, 129, 1, 1), (32, 4111, 1, 1), (20, 4111, 8, 8)]),
    ("dropout", False, (128,), True, [(128, 257, 2, 2), (2, 129, 1, 1), (300, 129, 1, 1)]),
    ("dropout", True, (64,), False, [(96, 129, 16, 16), (2, 129, 1, 1), (256, 129, 4, 4), (256, 257, 4, 4)]),
    ("dropout", True, (128,), False, [(96, 129, 16, 16), (2, 129, 1, 1), (40, 129, 4, 4)]),
    ("dropout", True, (64,), True, [(128, 129, 16, 16), (2, 129, 1, 1), (1, 4111, 32, 32), (160, 4111, 1, 1)]),
    ("dropout", True, (128,), True, [(96, 129, 16, 16), (2, 129, 1, 1), (300, 129, 1, 1)]),
    ("mask", False, (64, 128), False, [(3, 129, 32, 32), (2, 129, 1, 1)]),
    ("mask", False, (64, 128), True, [(256, 129, 1, 1), (2, 129, 1, 1)]),
    ("plain", False, (32, 48, 96, 120), False, [(40, 129, 4, 4), (2, 129, 1, 1)]),
    ("plain", False, (64,), False, [(96, 300, 1, 1), (300, 257, 1, 1), (2, 129, 1, 1), (1, 300, 1, 1), (96, 257, 2, 2), (300, 400, 1, 1), (2, 40, 1, 1)]),
    ("plain", False, (128,), False, [(5, 257, 16, 16), (2, 129, 1, 1), (40, 129, 2, 2), (40, 129, 4, 4)]),
    ("plain", False, (32, 48, 96, 120), True, [(128, 257, 2, 2), (2, 129, 1, 1)]),
    ("plain", False, (64,), True, [(300, 600, 1, 1), (2, 129, 1, 1), (1, 300, 1, 1), (96, 257, 2, 2), (16, 400, 32, 16), (2, 40, 1, 1), (32, 4111, 1, 1), (20, 4111, 8, 8)]),
    ("plain", False, (128,), True, [(128, 257, 2, 2), (2, 129, 1, 1), (3, 129, 32, 32)]),
    ("plain", True, (32, 48, 96, 120), False, [(96, 129, 16, 16), (2, 129, 1, 1)]),
    ("plain", True, (64,), False, [(400, 400, 2, 2), (160, 600, 4, 4), (1, 300, 1, 1), (160, 300, 4, 4)]),
    ("plain", True, (128,), False, [(96, 129, 16, 16), (2, 129, 1, 1), (1, 511, 32, 32)]),
    ("plain", True, (32, 48, 96, 120), True, [(96, 129, 16, 16), (2, 129, 1, 1)]),
    ("plain", True, (64,), True, [(1, 300, 1, 1), (96, 600, 8, 8), (160, 4111, 1, 1), (1, 4111, 32, 32)]),
    ("plain", True, (128,), True, [(96, 129, 16, 16), (2, 129, 1, 1), (5, 161, 32, 32)]),
    ("window", False, (64, 128), False, [(64, 257, 2, 2), (2, 129, 1, 1)]),
    ("window", True, (64, 128), False, [(96, 129, 16, 16), (2, 129, 1, 1)]),
]
WINDOW, P_DROP, SEED = (100, 30), 0.2, 78


def cases():
    return [(kind, packed, d, causal, *shape) for kind, packed, ds, causal, shapes in FORMS for d in ds for shape in shapes]


def lengths(nseq, longest):
    """Of a packed batch: the longest, and all kinds of shorter ones."""
    return [longest] + [1 + 37 * i % longest for i in range(1, nseq)]


def backward_call(kind, packed, d, causal, B, N, Hq, Hkv, f16):
    """For launches.launches."""
    lead, ws = [P] * (11 if kind in ("mask", "blocks") else 10), 1 << 40
    if packed:
        size = [P, B, sum(lengths(B, N)), N, Hq, Hkv, d, 0.1]
    else:
        size = [B, Hq, Hkv, N, N, d, 0.1]
    name = {"plain": ("fa_cross_bwd", "fa_varlen_bwd"), "window": ("fa_local_bwd", "fa_varlen_local_bwd"),
            "dropout": ("fa_dropout_bwd", "fa_varlen_dropout_bwd"), "mask": ("fa_mask_bwd",), "blocks": ("fa_blocksparse_bwd",)}[kind][packed]
    options = {"plain": [causal], "window": list(WINDOW), "dropout": [causal, P_DROP, SEED], "mask": [causal, 0, 0, (N + 7) // 8 * 8],
               "blocks": [causal, 64, 0, 0]}[kind]
    return name, lead + [ws] + size + options + [0, f16]
