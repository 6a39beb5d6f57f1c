"""The binding's two ways into cfgzip_decode_step and cfgzip_engine_step, the extension (plain tensors, the current
stream) and ctypes (a stream handed over, and everything else): the same results bit for bit, the same errors, the
stream that is current, and which calls go which way."""

import threading

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


def _by_extension(lib, step, args):
    """What the extension answers: a result, a status, or None for "not mine"."""
    return getattr(lib.binding, f"_{step}_step")(*args.values())


def _call(lib, step, args, **stream):
    keywords = {k: args[k] for k in KEYWORDS[step]}
    positional = [v for k, v in args.items() if k not in keywords]
    return getattr(lib, f"cfgzip_{step}_step")(*positional, **keywords, **stream)


def _bits(t):
    t = t.detach().contiguous()
    return t.view({4: torch.int32, 2: torch.int16}[t.element_size()]).cpu()


def _copy(args):
    return {k: v.clone() if isinstance(v, torch.Tensor) else v for k, v in args.items()}


def _same_both_ways(lib, step, args, wrap=lambda args: args):
    """Runs `args` by ctypes and, wrapped, as the binding decides; outputs must be the same bit for bit."""
    one, two = _copy(args), wrap(_copy(args))
    want, got = _call(lib, step, one, stream=torch.cuda.current_stream()), _call(lib, step, two)
    torch.cuda.synchronize()
    given = "rep_out" if step == "decode" else "states_out"
    if two[given] is not None:
        assert got is two[given] and want is one[given]
    assert got.shape == want.shape and got.dtype is want.dtype and torch.equal(got.cpu(), want.cpu())
    for k in ("logits", "tok_bits_out"):
        if one[k] is not None:
            assert torch.equal(_bits(one[k]), _bits(two[k])), k
    assert not torch.equal(_bits(one["logits"]), _bits(args["logits"]))  # (something has been masked)


def _outputs(step, args, given):
    B, V = args["logits"].shape[0], args["class_of_token"].numel()
    if given:
        args["tok_bits_out"] = torch.full((B, (V + 31) // 32), -1, dtype=torch.int32, device="cuda")
        args["rep_out" if step == "decode" else "states_out"] = torch.full((B,), -7, dtype=torch.int32, device="cuda")
    return args


@pytest.mark.parametrize("given", [False, True])
@pytest.mark.parametrize("dtype", [torch.bfloat16, torch.float32])
@pytest.mark.parametrize("step", ["decode", "engine"])
def test_the_same_results(lib, step, dtype, given):
    for B, V, stride in ((1, 1, 1), (1, 33, 40), (5, 1003, 1003), (17, 4096, 4160)):
        print(f"case {step} B={B} V={V} stride={stride}", flush=True)
        args = _outputs(step, MAKE[step](B, B=B, V=V, dtype=dtype, stride=stride), given)
        args["class_of_token"][0] = 0
        args["cls_bits" if step == "decode" else "state_mask"][:, 0] = -2  # (class 0 is masked)
        if stride != V:
            args["V"] = V
        assert _by_extension(lib, step, _copy(args)) is not None
        _same_both_ways(lib, step, args)


def test_forms_that_the_extension_takes(lib):
    args = _decode_args()
    args["tok"] = args["tok"].view(5, 1)  # as a sampler leaves it; the result is [B]
    assert _by_extension(lib, "decode", _copy(args)) is not None
    _same_both_ways(lib, "decode", args)
    args = _engine_args()
    args["tok_prev"] = args["sig_rep"] = None  # the first step
    assert _by_extension(lib, "engine", _copy(args)) is not None
    _same_both_ways(lib, "engine", args)


class _Tagged(torch.Tensor):
    pass


@pytest.mark.parametrize("step", ["decode", "engine"])
@pytest.mark.parametrize("form", ["subclass", "numpy C", "numpy V", "function mode"])
def test_forms_that_are_left_to_ctypes(lib, step, form):
    from torch.overrides import TorchFunctionMode
    args = MAKE[step]()
    args["V"] = args["class_of_token"].numel()

    def wrap(args):
        if form == "subclass":
            args["logits"] = args["logits"].as_subclass(_Tagged)
        elif form != "function mode":
            args[form[-1]] = np.int64(args[form[-1]])
        return args

    class Mode(TorchFunctionMode):
        def __torch_function__(self, func, types, args=(), kwargs=None):
            return func(*args, **(kwargs or {}))

    if form == "function mode":
        with Mode():
            assert _by_extension(lib, step, args) is None
            _same_both_ways(lib, step, args)
    else:
        assert _by_extension(lib, step, wrap(_copy(args))) is None
        _same_both_ways(lib, step, args, wrap)


def _wrong(step):
    """(what is wrong, its change to the arguments)"""
    state = "cls_bits" if step == "decode" else "state_mask"
    ids = "tok" if step == "decode" else "states_in"

    def put(**changes):
        return lambda args: args.update({k: f(args[k]) for k, f in changes.items()})
    yield "logits on the CPU", put(logits=lambda t: t.cpu())
    yield "half logits", put(logits=lambda t: t.half())
    yield "logits of three dimensions", put(logits=lambda t: t[None])
    yield "a column stride", put(logits=lambda t: t[:, ::2])
    yield "64-bit masks", put(**{state: lambda t: t.long()})
    yield "masks on the CPU", put(**{state: lambda t: t.cpu()})
    yield "masks with a stride", put(**{state: lambda t: torch.cat([t, t], 1)[:, ::2]})
    yield "64-bit ids", put(**{ids: lambda t: t.long()})
    yield "64-bit class ids", put(class_of_token=lambda t: t.long())
    yield "token masks of another type", put(tok_bits_out=lambda t: torch.zeros((5, 32), dtype=torch.int64, device="cuda"))
    yield "more columns than a row has", put(V=lambda v: 1003, logits=lambda t: t[:, :900].contiguous())
    yield "no classes", put(C=lambda c: 0)
    yield "negative V", put(V=lambda v: -1)
    if step == "decode":
        yield "a mask row too few", put(cls_bits=lambda t: t[:-1])
        yield "a representative too many", put(rep_of_class=lambda t: torch.cat([t, t[:1]]))
        yield "a class id too few", put(class_of_token=lambda t: t[:-1])
        yield "a token too few", put(tok=lambda t: t[:-1])
        yield "representatives of another type", put(rep_out=lambda t: torch.zeros(5, device="cuda"))
    else:
        yield "32-bit signatures", put(sig_rep=lambda t: t.int())
        yield "tokens without signatures", put(sig_rep=lambda t: None)
        yield "states in place", lambda args: args.update(states_out=args["states_in"])
        yield "states of another type", put(states_out=lambda t: torch.zeros(5, device="cuda"))


@pytest.mark.parametrize("step,what", [(s, w) for s in MAKE for w, _ in _wrong(s)])
def test_the_same_errors(lib, step, what):
    """Every case is turned down before a kernel is launched."""
    print(f"case {step}: {what}", flush=True)
    args = MAKE[step]()
    dict(_wrong(step))[what](args)
    before = args["logits"].clone()
    said = []
    for stream in ({"stream": torch.cuda.current_stream()}, {}):
        with pytest.raises((ValueError, TypeError, IndexError, lib.CfgzipError)) as e:
            _call(lib, step, args, **stream)
        said.append((type(e.value), str(e.value)))
    assert said[0] == said[1]
    torch.cuda.synchronize()
    assert torch.equal(args["logits"], before)


@pytest.mark.parametrize("step", ["decode", "engine"])
def test_a_status_of_the_library_is_raised(lib, step):
    args = MAKE[step]()
    args["logits"], args["V"] = args["logits"][:, :900].contiguous(), 1003
    assert _by_extension(lib, step, args) == -1
    with pytest.raises(lib.CfgzipError):
        _call(lib, step, args)


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


@pytest.mark.parametrize("step", ["decode", "engine"])
def test_on_the_current_stream(lib, step):
    """The call comes behind what the current stream has been given before, a wait and the logits themselves, and not
    before it on another stream."""
    args = MAKE[step](B=16, V=30_001)
    want = _copy(args)
    out = _call(lib, step, want, stream=torch.cuda.current_stream())
    source = args["logits"].clone()
    args["logits"].zero_()
    assert _by_extension(lib, step, _copy(args)) is not None
    torch.cuda.synchronize()
    side = torch.cuda.Stream()
    with torch.cuda.stream(side):
        torch.cuda._sleep(20_000_000)
        args["logits"].copy_(source)
        got = _call(lib, step, args)
    side.synchronize()
    assert torch.equal(_bits(args["logits"]), _bits(want["logits"])) and torch.equal(got.cpu(), out.cpu())


def test_from_two_host_threads(lib):
    """A thread for each step, each on a stream of its own."""
    errors = []

    def work(step, seed):
        try:
            args = MAKE[step](seed, B=8, V=20_011)
            want = _copy(args)
            out = _call(lib, step, want, stream=torch.cuda.current_stream())
            torch.cuda.synchronize()
            with torch.cuda.stream(torch.cuda.Stream()) as _:
                for _ in range(50):
                    mine = _copy(args)
                    got = _call(lib, step, mine)
                    if not torch.equal(got.cpu(), out.cpu()) or not torch.equal(_bits(mine["logits"]), _bits(want["logits"])):
                        errors.append((step, "differs"))
        except Exception as e:  # noqa: BLE001 - reported by the main thread
            errors.append((step, repr(e)))

    threads = [threading.Thread(target=work, args=(s, k)) for k, s in enumerate(("decode", "engine", "decode", "engine"))]
    for t in threads:
        t.start()
    for t in threads:
        t.join(timeout=60)
    assert not any(t.is_alive() for t in threads)
    assert not errors, errors[:3]
