"""The binding's two ways into cfgzip_decode_step and cfgzip_engine_step, the extension (plain tensors, the current
stream) and ctypes (a stream handed over, and everything else): the same results bit for bit, the same errors, the
stream that is current, and which calls go which way."""

import numpy as np
import pytest

from gpu_util import dev

pytestmark = pytest.mark.gpu

torch = pytest.importorskip("torch")


@pytest.fixture(scope="module")
def lib():
    import paper_2605_29986_amd as p
    p.load_library()
    assert p.binding._decode_step.__module__ == "cfgzip_stepcall"
    return p


def _logits(rng, B, stride, dtype):
    return torch.from_numpy(rng.standard_normal((B, stride), dtype=np.float32)).cuda().to(dtype)


def _decode_args(seed=0, B=5, V=1003, C=77, dtype=torch.bfloat16, stride=None):
    rng = np.random.default_rng(seed)
    return {"logits": _logits(rng, B, stride or V, dtype),
            "cls_bits": dev(rng.integers(0, 1 << 32, size=(B, (C + 31) // 32), dtype=np.uint32)),
            "class_of_token": dev(rng.integers(0, C, size=V).astype(np.int32)), "C": C,
            "tok": dev(rng.integers(0, V, size=B).astype(np.int32)),
            "rep_of_class": dev(rng.integers(0, V, size=C).astype(np.int32)),
            "tok_bits_out": None, "rep_out": None, "V": None}


def _engine_args(seed=0, B=5, V=1003, C=77, S=31, dtype=torch.float32, stride=None):
    rng = np.random.default_rng(seed)
    return {"logits": _logits(rng, B, stride or V, dtype),
            "state_mask": dev(rng.integers(0, 1 << 32, size=(S, (C + 31) // 32), dtype=np.uint32)), "C": C,
            "class_of_token": dev(rng.integers(0, C, size=V).astype(np.int32)),
            "sig_rep": dev(rng.integers(0, S, size=(C, S)).astype(np.uint16)),
            "tok_prev": dev(rng.integers(0, V, size=B).astype(np.int32)),
            "states_in": dev(rng.integers(0, S, size=B).astype(np.int32)),
            "states_out": None, "tok_bits_out": None, "V": None}


MAKE = {"decode": _decode_args, "engine": _engine_args}
KEYWORDS = {"decode": ("tok_bits_out", "rep_out", "V"), "engine": ("states_out", "tok_bits_out", "V")}


def _call(lib, step, args, **stream):
    keywords = {k: args[k] for k in KEYWORDS[step]}
    positional = [v for k, v in args.items() if k not in keywords]
    return getattr(lib, f"cfgzip_{step}_step")(*positional, **keywords, **stream)


@pytest.mark.parametrize("step", ["decode", "engine"])
def test_what_a_dispatch_mode_raises(lib, step):
    """An error out of Python below the allocation of the result is that error, and nothing is launched."""
    from torch.utils._python_dispatch import TorchDispatchMode

    class Refuses(TorchDispatchMode):
        def __torch_dispatch__(self, func, types, args=(), kwargs=None):
            raise ZeroDivisionError(str(func))

    args = MAKE[step]()
    before = args["logits"].clone()
    for stream in ({"stream": torch.cuda.current_stream()}, {}):
        with pytest.raises(ZeroDivisionError, match="empty"), Refuses():
            _call(lib, step, args, **stream)
    torch.cuda.synchronize()
    assert torch.equal(args["logits"], before)
