"""The calls of the pre-computation through the binding's extension and through ctypes: the same results and the same
errors."""

import numpy as np
import pytest

from synthetic_inputs.dfa import make_lexer_dfa
from synthetic_inputs.grammar import make_json_gnf
from synthetic_inputs.nfa import add_transitions, nfa_from_dfa
from synthetic_inputs.vocab import make_vocab_mixture

pytestmark = pytest.mark.gpu

torch = pytest.importorskip("torch")

S, V = 160, 700


@pytest.fixture(scope="module")
def lib():
    import paper_2605_29986_amd as p
    p.load_library()
    return p


def _bytes(n):
    return torch.zeros(max(int(n), 256), dtype=torch.uint8, device="cuda")


def _calls(lib):
    """{name: (function, positional arguments, keyword arguments)}, each of the plain form that the extension takes."""
    raw = lib.load_library()
    table, keywords = make_lexer_dfa(3, S)
    v = make_vocab_mixture(4, V, 16, 0.0, keywords)
    tb, to, tt = (torch.from_numpy(x).cuda() for x in (v.tok_bytes, v.tok_off, table))
    nfa = torch.from_numpy(add_transitions(nfa_from_dfa(table), 5, 0.1).view(np.int32)).cuda()
    g = make_json_gnf()
    gd = [torch.from_numpy(x).cuda() for x in g.arrays()]
    ws_sig = _bytes(raw.cfgzip_signatures_workspace_bytes(V, S))
    sig, h = lib.cfgzip_signatures(tb, to, tt, workspace=ws_sig, stream=torch.cuda.current_stream())

    def room(*shape, dtype=torch.int32):
        return torch.empty(shape, dtype=dtype, device="cuda")

    return {
        "signatures": (lib.cfgzip_signatures, [tb, to, tt], {"workspace": _bytes(ws_sig.numel())}),
        "hashes": (lib.cfgzip_signatures, [tb, to, tt], {"workspace": _bytes(ws_sig.numel()), "want_sig": False, "hash_seed": -7}),
        "signatures into": (lib.cfgzip_signatures, [tb, to, tt],
                            {"workspace": _bytes(ws_sig.numel()), "sig_out": room(V, S, dtype=torch.uint16),
                             "hash_out": room(V, dtype=torch.int64)}),
        "hashes into": (lib.cfgzip_signatures, [tb, to, tt], {"workspace": _bytes(ws_sig.numel()), "want_sig": False,
                                                              "hash_out": room(V, dtype=torch.int64)}),
        "classes": (lib.cfgzip_build_classes, [tb, to, tt, sig, h],
                    {"workspace": _bytes(raw.cfgzip_build_classes_workspace_bytes(V, S)), "signatures_workspace": ws_sig}),
        "rows": (lib.cfgzip_build_classes, [tb, to, None, sig, h],
                 {"workspace": _bytes(raw.cfgzip_build_classes_workspace_bytes(V, S)),
                  "rep_of_class": room(V)}),
        "classes into": (lib.cfgzip_build_classes, [tb, to, tt, sig, h],
                         {"workspace": _bytes(raw.cfgzip_build_classes_workspace_bytes(V, S)), "class_of_token": room(V),
                          "rep_of_class": room(V)}),
        "displacements": (lib.cfgzip_displacements, [tb, to, *gd, g.N],
                          {"workspace": _bytes(raw.cfgzip_displacements_workspace_bytes(V, g.N, g.P)), "row_len": 512}),
        "nfa": (lib.cfgzip_nfa_signatures, [tb, to, nfa], {}),
    }


ENTRIES = {"signatures": "_signatures", "hashes": "_signatures", "signatures into": "_signatures", "hashes into": "_signatures",
           "classes": "_build_classes", "rows": "_build_classes", "classes into": "_build_classes",
           "displacements": "_displacements", "nfa": "_nfa_signatures"}
NAMES = list(ENTRIES)
INTO = ("sig_out", "hash_out", "class_of_token", "rep_of_class")


def _plain(out):
    return [x.cpu().numpy().tobytes() if torch.is_tensor(x) else x for x in out]


def _outcome(f, args, kw):
    try:
        return _plain(f(*args, **kw))
    except Exception as e:  # noqa: BLE001 - which one is what is compared
        return type(e), str(e)


def _wipe(kw):
    """What a call is to write holds something else before it."""
    for name in INTO:
        if name in kw:
            kw[name].view(torch.uint8).fill_(0xA5)


@pytest.mark.parametrize("name", NAMES)
def test_the_same_results(lib, name, monkeypatch):
    from paper_2605_29986_amd import binding
    f, args, kw = _calls(lib)[name]
    taken = []
    plain = getattr(binding, ENTRIES[name])
    monkeypatch.setattr(binding, ENTRIES[name], lambda *a: taken.append(plain(*a)) or taken[-1])
    results = []
    for stream in ({}, {"stream": torch.cuda.current_stream()}):
        _wipe(kw)
        out = f(*args, **kw, **stream)
        # read before the next call writes the same tensors
        results.append((out, _plain(out), [(x.dtype, x.shape, x.device) if torch.is_tensor(x) else type(x) for x in out]))
        for given in INTO:
            if given in kw:
                assert any(torch.is_tensor(x) and x.data_ptr() == kw[given].data_ptr() for x in out), given
    assert len(taken) == 1 and taken[0] is not None and type(taken[0]) is not int
    (_, by_extension, kinds), (_, by_ctypes, other_kinds) = results
    assert by_extension == by_ctypes and kinds == other_kinds


@pytest.mark.parametrize("name", NAMES)
def test_the_current_stream(lib, name):
    """On a side stream, behind work that has the inputs ready late: a call elsewhere would read what was there before."""
    f, args, kw = _calls(lib)[name]
    _wipe(kw)
    want = _plain(f(*args, **kw, stream=torch.cuda.current_stream()))
    tables = [i for i, x in enumerate(args) if torch.is_tensor(x) and x.dtype is not torch.int64]
    ready = [args[i].clone() for i in tables]
    if name in ("classes", "classes into"):
        tables, ready = [], []  # (what the signature call has put by stays as it is: the hashes and rows come late)
    late = [i for i, x in enumerate(args) if name in ("classes", "classes into", "rows") and torch.is_tensor(x) and i in (3, 4)]
    ready += [args[i].clone() for i in late]
    tables += late
    _wipe(kw)
    for i in tables:
        args[i].view(torch.uint8).zero_()
    torch.cuda.synchronize()
    side = torch.cuda.Stream()
    with torch.cuda.stream(side):
        torch.cuda._sleep(20_000_000)  # some ms
        for i, x in zip(tables, ready):
            args[i].view(torch.uint8).copy_(x.view(torch.uint8))
        out = f(*args, **kw)
        side.synchronize()
        assert _plain(out) == want


@pytest.mark.parametrize("name", NAMES)
def test_the_same_errors(lib, name):
    """Every tensor in turn of another type, in host memory, not contiguous, or no tensor; a workspace too small."""
    f, args, kw = _calls(lib)[name]
    stream = {"stream": torch.cuda.current_stream()}
    wrongs = [lambda x: x.cpu(), lambda x: x.float(), lambda x: torch.stack([x, x], -1)[..., 0], lambda x: 5, lambda x: None]
    for i, x in enumerate(args):
        if not torch.is_tensor(x):
            continue
        for wrong in wrongs:
            bad = [*args[:i], wrong(x), *args[i + 1:]]
            if name in ("classes", "rows", "classes into") and (i == 3 or i == 2) and bad[i] is None:
                continue  # other calls, that may be right
            assert _outcome(f, bad, kw) == _outcome(f, bad, {**kw, **stream}), (i, wrong(x))
    if "workspace" in kw:
        small = {**kw, "workspace": _bytes(256)}
        got = _outcome(f, args, small)
        assert got == _outcome(f, args, {**small, **stream}) and got[0] is lib.CfgzipError
