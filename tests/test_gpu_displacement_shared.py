"""GPU parity of the shared walk of cfgzip_displacements where it can go wrong: vocabulary sizes around its waves
and workgroups, sets of one and two configurations a lane and of more than it takes, grammars whose productions or
relation do not fit its LDS, bytes with equal productions, rows that are only 8-byte aligned, and vocabularies that
exhaust its tables, so that some tokens are taken alone by the passes behind it.  Compared like every other
displacement: status, row and hash of every token against the oracle, and the classes."""

import ctypes
import itertools

import numpy as np
import pytest

from oracle import displacement as D
from synthetic_inputs.grammar import (grammar_from_productions, make_bracket_gnf, make_json_gnf, make_random_gnf,
                                      make_token_strings)
from synthetic_inputs.vocab import vocab_from_tokens
from test_gpu_displacement import _check_adjacency, _check_rows, _grammar_dev

pytestmark = pytest.mark.gpu

torch = pytest.importorskip("torch")


@pytest.fixture(scope="module")
def lib():
    import paper_2605_29986_amd as p
    p.load_library()
    return p


@pytest.mark.parametrize("V", [1, 15, 16, 17, 255, 4095, 4097])
def test_vocabulary_sizes(lib, V):
    print(f"case V={V}", flush=True)
    g, atoms = make_bracket_gnf(3)
    _check_rows(lib, g, make_token_strings(V, V, atoms + b"()[]{},+", 9))


@pytest.mark.parametrize("n", [63, 64, 65, 100, 127, 128, 129, 200])
def test_sets_of_many_configurations(lib, n):
    """n alternatives for the first byte, all of them alive after every further one; on 'b' every second goes."""
    print(f"case n={n}", flush=True)
    prods = [(A, ord("a"), (A,)) for A in range(n)] + [(A, ord("b"), (A,)) for A in range(0, n, 2)]
    prods += [(A, ord("c"), ()) for A in range(n)]
    g = grammar_from_productions(n, prods)
    vocab = vocab_from_tokens([b"", b"a", b"aa", b"ab", b"aab", b"aba", b"abb", b"ac", b"acc", b"c", b"cc", b"b", b"z"])
    _check_rows(lib, g, vocab, row_len=1024)


@pytest.mark.parametrize("n_nt,n_prod", [(40, 1023), (40, 1024), (40, 1025), (128, 900), (129, 900), (200, 1100),
                                         (255, 700), (256, 700)])
def test_grammars_around_what_is_kept_in_lds(lib, n_nt, n_prod):
    print(f"case N={n_nt} P={n_prod}", flush=True)
    alphabet = bytes(range(97, 123)) + b"0123456789"
    g = make_random_gnf(n_nt + n_prod, n_nt, alphabet, n_prod, 5)
    _check_adjacency(lib, g)
    _check_rows(lib, g, make_token_strings(7, 300, alphabet, 5), row_len=512)


@pytest.mark.parametrize("n", [62, 63, 64, 65, 100, 129])
def test_many_productions_of_one_symbol_and_byte(lib, n):
    """Up to 63 productions of a (byte, symbol) pair are looked up together; with more of one pair, none are.  The pair lies
    first, last and between others among the productions of its byte."""
    print(f"case n={n}", flush=True)
    for head in (0, n // 2, n + 1):
        prods = [(head, ord("a"), (B,)) for B in range(n)] + [(A, ord("a"), ()) for A in range(n + 2) if A != head]
        prods += [(A, ord("b"), (head,)) for A in range(0, n + 2, 3)] + [(A, ord("c"), ()) for A in range(1, n + 2, 40)]
        g = grammar_from_productions(n + 2, prods)
        vocab = vocab_from_tokens([bytes(w) for k in range(4) for w in itertools.product(b"abc", repeat=k)] + [b"z", b"az"])
        _check_rows(lib, g, vocab, row_len=1024)


@pytest.mark.parametrize("n", [31, 32, 33])
def test_productions_of_a_byte_around_a_bit_each(lib, n):
    """Up to 32 productions of a byte are told by a bit each: pops of the first and the last of them, of runs of one symbol,
    and backtracks that all, some or none of them may take."""
    print(f"case n={n}", flush=True)
    prods = [(A, ord("a"), (A, (A + 1) % n)) for A in range(n)] + [(0, ord("b"), (B,)) for B in range(n)]
    prods += [(n - 1, ord("c"), ())] + [(A, ord("d"), ()) for A in range(0, n, 3)] + [(1, ord("d"), (B,)) for B in (0, n - 1)]
    g = grammar_from_productions(n, prods)
    vocab = vocab_from_tokens([bytes(w) for k in range(4) for w in itertools.product(b"abcd", repeat=k)] + [b"z", b"ddddd"])
    _check_rows(lib, g, vocab, row_len=1024)


@pytest.mark.parametrize("own", [31, 32, 33])
def test_pairs_of_byte_and_symbol_around_what_is_kept(lib, own):
    """62 symbols and two entries more for each of `own` bytes: up to 2,048 are kept."""
    print(f"case own={own}", flush=True)
    rng = np.random.default_rng(own)
    prods = [(A, 40 + (A * 7) % own, ()) for A in range(62)]
    prods += [(int(rng.integers(0, 62)), 40 + b, tuple(int(x) for x in rng.integers(0, 62, size=int(rng.integers(1, 4)))))
              for b in range(own) for _ in range(3)]
    g = grammar_from_productions(62, sorted(set(prods)))
    _check_rows(lib, g, make_token_strings(own, 900, bytes(range(40, 40 + own)) + b"~", 5), row_len=512)


def test_records_that_differ_late(lib):
    """Queues and stacks of equal lengths whose first eight and more symbols are alike, in sets of a few and of more than 64
    records, and bodies of more than four symbols among short ones."""
    n = 40
    prods = [(0, ord("a"), ())] + [(k, ord("b"), ()) for k in range(1, n)] + [(n, ord("s"), (0, k)) for k in range(n)]
    prods += [(n + 1, ord("q"), (n + 1, 0, 0, 0)), (n + 1, ord("r"), ())]
    prods += [(n + 2, ord("x"), (n + 1, j)) for j in range(1, 6)] + [(n + 2, ord("y"), (n + 1, 0, j)) for j in range(1, n)]
    prods += [(n + 2, ord("y"), (n + 1, 1, j)) for j in range(1, n)] + [(n + 2, ord("y"), (n + 1, 1, 2, 3, 4, j)) for j in (7, 8)]
    g = grammar_from_productions(n + 3, sorted(set(prods)))
    toks = [b"a" * k + t for k in range(0, 14) for t in (b"", b"b", b"ba")]
    toks += [h + b"q" * k + t for h in (b"x", b"y") for k in range(6) for t in (b"", b"r", b"raa", b"raab")]
    _check_rows(lib, g, vocab_from_tokens(toks), row_len=4096)


def test_bytes_with_equal_productions(lib):
    """Digits 0-4 behave alike, 5 differs in a body, 6 in the fifth symbol of a long one, 7 in the number of
    productions."""
    prods = [(0, d, (1, 2)) for d in b"01234567"] + [(1, d, (2, 2, 2, 2, 2)) for d in b"012345"]
    prods += [(1, ord("6"), (2, 2, 2, 2, 1)), (1, ord("7"), (2, 2, 2, 2, 2)), (2, ord("7"), (0,))]
    prods += [(2, d, ()) for d in b"012346"] + [(2, ord("5"), (1,)), (2, ord("7"), ())]
    g = grammar_from_productions(3, prods)
    _check_rows(lib, g, make_token_strings(1, 600, b"012345678", 5), row_len=1024)


def test_vocabulary_that_exhausts_the_tables(lib):
    """Every symbol may follow every other, so a token's queue is the token itself: every prefix of every token is a
    set of its own."""
    n = 26
    prods = [(A, 97 + A, ()) for A in range(n)] + [(n, 65, (A, B)) for A in range(n) for B in range(n)]
    g = grammar_from_productions(n + 1, prods)
    rng = np.random.default_rng(2)
    toks = [bytes(rng.integers(97, 123, size=int(k), dtype=np.uint8)) for k in rng.integers(24, 36, size=12_000)]
    _check_rows(lib, g, vocab_from_tokens(toks), expect_overflow=True)


def test_deep_stacks_behind_exhausted_tables(lib):
    """Tokens of a few random symbols (no sets are shared) and then a stack that grows by two with every byte: queues and
    stacks on both sides of what the passes behind the shared walk hold."""
    n = 26
    prods = [(A, 97 + A, ()) for A in range(n)] + [(n, 64, (A, B)) for A in range(n) for B in range(n)]
    prods += [(n, 64, (A, n + 1)) for A in range(n)] + [(n + 1, ord("+"), (n + 1,) * 3), (n + 1, ord("-"), ())]
    g = grammar_from_productions(n + 2, prods)
    rng = np.random.default_rng(3)
    toks = [bytes(rng.integers(97, 123, size=int(k), dtype=np.uint8)) + b"+" * int(p) + b"-" * int(m)
            for k, p, m in zip(rng.integers(8, 28, size=9_000), rng.integers(0, 18, size=9_000), rng.integers(0, 4, size=9_000))]
    _check_rows(lib, g, vocab_from_tokens(toks), expect_overflow=True)


def test_rounds_of_more_bytes_than_are_staged(lib):
    """Single tokens around 256 bytes and of 700, and a third of a vocabulary of 80 to 140 among tokens of a few bytes.
    (A workgroup keeps up to 6,144 bytes of a batch in LDS, which none of these comes to: see below.)"""
    g = grammar_from_productions(1, [(0, ord("a"), (0,)), (0, ord("a"), ()), (0, ord("b"), (0,))])
    rng = np.random.default_rng(5)
    long_ones = [b"ab" * 127 + b"a", b"ab" * 128, b"ab" * 128 + b"a", b"a" * 700, b"b" * 255 + b"z" + b"a" * 40]
    _check_rows(lib, g, vocab_from_tokens(long_ones))
    toks = [bytes(rng.integers(97, 99, size=int(m), dtype=np.uint8))
            for m in np.where(rng.random(9_000) < 0.3, rng.integers(80, 140, size=9_000), rng.integers(0, 5, size=9_000))]
    _check_rows(lib, g, vocab_from_tokens(toks + long_ones))


@pytest.mark.parametrize("n", [26, 120])
def test_tokens_that_share_no_sets(lib, n):
    """Sets of one configuration that a lane works out alone, after its wave has worked out a few: pops, backtracks on
    an empty stack, bodies of none to six symbols, bytes that nothing applies to, and lists past their bound."""
    rng = np.random.default_rng(n)
    prods = [(A, 97 + A % 26, ()) for A in range(n)]                                          # pop, one or more per byte
    prods += [(A, 65 + (A + 7) % 26, tuple(int(x) for x in rng.integers(0, n, size=A % 7))) for A in range(n)]
    prods += [(n, 35, (A, B)) for A in range(min(n, 26)) for B in range(min(n, 26))]          # any may follow any of these
    g = grammar_from_productions(n + 1, prods)
    alphabet = np.frombuffer(b"abcdefghijklmnopqrstuvwxyzABCDEFGHIJKLMNOPQRSTUVWXYZ", np.uint8)
    toks = [bytes(alphabet[rng.integers(0, 26 if k % 3 else 52, size=int(m))])
            for k, m in enumerate(rng.integers(1, 10, size=9_000))]
    toks += [b"ab!cd", b"!", b"a" * 33, b"ab" * 20, b"#ab", b"abc#"] * 8
    _check_rows(lib, g, vocab_from_tokens(toks))


def test_rows_that_are_only_8_byte_aligned(lib):
    from gpu_util import dev
    g = make_json_gnf()
    vocab = make_token_strings(4, 500, b'{}[]:,"0123456789tfnrue ', 8)
    tb, to, gd = dev(vocab.tok_bytes), dev(vocab.tok_off), _grammar_dev(g)
    want, want_hash, want_status = lib.cfgzip_displacements(tb, to, *gd, g.N)
    raw = lib.load_library()
    buf = torch.full((vocab.V * 256 + 8,), 7, dtype=torch.int16, device="cuda")
    h = torch.empty(vocab.V, dtype=torch.int64, device="cuda")
    st = torch.empty(vocab.V, dtype=torch.int32, device="cuda")
    ws = torch.empty(raw.cfgzip_displacements_workspace_bytes(vocab.V, g.N, g.P), dtype=torch.uint8, device="cuda")
    rc = raw.cfgzip_displacements(tb.data_ptr(), to.data_ptr(), vocab.V, *[x.data_ptr() for x in gd], gd[3].numel(),
                                  g.P, g.N, buf.data_ptr() + 8, 256, h.data_ptr(), st.data_ptr(),
                                  ctypes.c_uint64(lib.DEFAULT_HASH_SEED), ws.data_ptr(), ws.numel(),
                                  torch.cuda.current_stream().cuda_stream)
    assert rc == 0
    got = buf.cpu().numpy()
    assert (got[4:-4].reshape(vocab.V, 256) == want.view(torch.int16).cpu().numpy()).all()
    assert (got[:4] == 7).all() and (got[-4:] == 7).all()
    assert torch.equal(h, want_hash) and torch.equal(st, want_status)


STAGED = 6144  # bytes of a batch's tokens that a workgroup keeps in LDS


def _batch_bytes(off, n_cu):
    """The bytes of every batch of up to 1,024 tokens, workgroup after workgroup."""
    V = len(off) - 1
    per_group = -(-V // min(n_cu, -(-V // 16)))
    return [[int(off[min(b + 1024, g + per_group, V)] - off[b]) for b in range(g, min(g + per_group, V), 1024)]
            for g in range(0, V, per_group)]


def _n_cu():
    return torch.cuda.get_device_properties(0).multi_processor_count


@pytest.mark.parametrize("total", [STAGED - 1, STAGED, STAGED + 1, 20_000])
@pytest.mark.parametrize("V", [1, 2, 16])
def test_bytes_around_what_is_staged(lib, V, total):
    """One workgroup whose tokens have so many bytes together; beyond what is staged they are read from memory.  Every
    byte permutes five symbols, so a token's set says all of its bytes' product."""
    from gpu_util import dev, hash_np
    print(f"case V={V} total={total}", flush=True)
    rng = np.random.default_rng(total + V)
    g = grammar_from_productions(5, [(A, b, (int(B),)) for b in b"abcd" for A, B in enumerate(rng.permutation(5))])
    ends = np.sort(rng.integers(0, total + 1, size=V - 1))
    data = rng.integers(97, 101, size=total, dtype=np.uint8).tobytes()
    vocab = vocab_from_tokens([data[a:b] for a, b in zip([0, *ends], [*ends, total])])
    assert _batch_bytes(vocab.tok_off, _n_cu()) == [[total]]
    rows, hashes, status = lib.cfgzip_displacements(dev(vocab.tok_bytes), dev(vocab.tok_off), *_grammar_dev(g), g.N, hash_seed=9)
    prods = g.productions()
    for t, tok in enumerate(vocab.tokens()):
        # (step by step: Algorithm 1's recursion goes as deep as the token is long)
        row, h, st = D.encode_displacement(D.displacement_within_limits(tuple(tok), prods, D.stack_adjacency(prods)), t, 9, 256)
        assert st == D.DISP_OK == int(status[t]) and int(hash_np(hashes)[t]) == h
        assert (rows[t].cpu().numpy() == np.asarray(row, np.uint16)).all()


def _check_repeated(lib, g, few, pick):
    """The vocabulary of the strings few[pick]: every row, hash and status are its string's (and those the oracle's)."""
    _check_rows(lib, g, few, expect_overflow=None)
    strings = few.tokens()
    vocab = vocab_from_tokens([strings[i] for i in pick])
    gd = _grammar_dev(g)

    def run(v):
        return lib.cfgzip_displacements(torch.from_numpy(v.tok_bytes).cuda(), torch.from_numpy(v.tok_off).cuda(), *gd, g.N,
                                        row_len=256)

    rows, h, status = run(few)
    many_rows, many_h, many_status = run(vocab)
    p = torch.from_numpy(pick).cuda()
    assert bool((many_status == status[p]).all())
    ok = many_status == 0  # a token that overflows has a row and a hash of its own
    assert bool(ok.any())
    assert bool((many_h == h[p])[ok].all())
    for a in range(0, vocab.V, 1 << 16):
        part = slice(a, min(vocab.V, a + (1 << 16)))
        same = (many_rows[part].view(torch.int16) == rows.view(torch.int16)[p[part]]).all(dim=1)
        assert bool(same[ok[part]].all())
    return vocab


def test_staged_and_unstaged_batches_one_after_the_other(lib):
    """Workgroups of 1,100 tokens, a batch of 1,024 and one of 76: both with their bytes in LDS, either one, and neither."""
    n_cu, per_group = _n_cu(), 1100
    rng = np.random.default_rng(8)
    few = vocab_from_tokens([bytes(rng.integers(97, 100, size=int(m), dtype=np.uint8)) for m in rng.integers(0, 5, size=300)]
                            + [bytes(rng.integers(97, 99, size=int(m), dtype=np.uint8)) for m in rng.integers(90, 130, size=80)])
    pick = rng.integers(0, 300, size=(n_cu, per_group))
    for g in range(n_cu):
        if g & 1:
            pick[g, rng.choice(1024, size=70, replace=False)] = rng.integers(300, few.V, size=70)
        if g & 2:
            pick[g, 1024:] = rng.integers(300, few.V, size=per_group - 1024)
    g = grammar_from_productions(5, [(A, b, (int(B),)) for b in b"abc" for A, B in enumerate(rng.permutation(5))])
    vocab = _check_repeated(lib, g, few, pick.ravel())
    kinds = {(first > STAGED, second > STAGED) for first, second in _batch_bytes(vocab.tok_off, n_cu)}
    assert len(kinds) == 4


@pytest.mark.parametrize("V,longest", [(16_384, 6), (16_385, 6), (32_768, 6), (32_769, 6), (33_100, 80), (65_536, 5),
                                       (65_537, 5), (262_144, 4), (262_401, 4)])
def test_groups_around_the_sorted_batches(lib, V, longest):
    """64 tokens for a workgroup, which its waves take at once, and 65, which are sorted by length; 256 and 257, of which a wave
    takes more at a time; tokens of up to 80 bytes;
    a whole batch of 1,024 tokens and one more.  The vocabulary repeats 700 strings: theirs are compared with the oracle, and
    every row, hash and status with its string's."""
    print(f"case V={V} longest={longest}", flush=True)
    few = make_token_strings(V, 700, b'{}[]",:0123456789.eE+-truefalsn \\ua', longest)
    _check_repeated(lib, make_json_gnf(), few, np.random.default_rng(V).integers(0, few.V, size=V))


def _hard_grammar(n):
    """The JSON grammar, and n bytes that stand for a symbol each, which may all follow each other: every string of those is
    a queue of its own.  The grammar and the bytes."""
    json = make_json_gnf()
    taken = {int(b) for b in json.byte}
    free = [b for b in range(1, 32) if b not in taken]
    own, pairs = free[:n], free[n:2 * n]
    prods = json.productions()
    for i in range(n):
        prods.append((json.N + i, own[i], ()))
        prods += [(json.N + n, pairs[i], (json.N + i, json.N + j)) for j in range(n)]
    return grammar_from_productions(json.N + n + 1, prods), own


def _call_us(lib, g, vocab, row_len):
    gd = _grammar_dev(g)
    tb, to = torch.from_numpy(vocab.tok_bytes).cuda(), torch.from_numpy(vocab.tok_off).cuda()
    times = []
    for _ in range(7):
        begin, end = torch.cuda.Event(enable_timing=True), torch.cuda.Event(enable_timing=True)
        begin.record()
        lib.cfgzip_displacements(tb, to, *gd, g.N, row_len=row_len)
        end.record()
        end.synchronize()
        times.append(begin.elapsed_time(end) * 1e3)
    return sorted(times)[3]


def test_tokens_that_share_no_sets_side_by_side(lib):
    """300 tokens behind each other that one workgroup has no room for, most of which need the widest caps: their results, and
    that the whole chip takes part.  (Three times what the same tokens take spread over the vocabulary, whose walks have room
    for them; 38 times with one workgroup at work.)"""
    g, own = _hard_grammar(9)
    rng = np.random.default_rng(12)
    easy = make_token_strings(31, 400, b'{}[]",:0123456789.eE+-truefalsn \\ua', 8).tokens()
    hard = [bytes(own[i] for i in rng.integers(0, 9, size=28)) for _ in range(300)]
    few = vocab_from_tokens(easy + hard)
    pick = np.concatenate([rng.integers(0, 400, size=120_000), np.arange(400, 700)])
    vocab = _check_repeated(lib, g, few, pick)
    spread = vocab_from_tokens([few.token(i) for i in rng.permutation(pick)])
    together, apart = _call_us(lib, g, vocab, 256), _call_us(lib, g, spread, 256)
    print(f"together {together:.0f} us, apart {apart:.0f} us", flush=True)
    assert together < 12 * apart


def test_room_for_sets_with_many_successors_alike(lib):
    """Sets of eight configurations with 64 successors of which eight are different: the tokens fit the shared walk's room (the
    second word of the workspace says how many did not; room for all successors was there for 12,000 of the 32,000)."""
    top, first, alike, marks = 0, 1, range(2, 10), range(10, 14)
    prods = [(first, ord("a"), (t,)) for t in alike] + [(t, ord("y"), (top,)) for t in alike]
    prods += [(top, ord("0") + i, (t, m)) for i, m in enumerate(marks) for t in alike] + [(m, ord("v"), ()) for m in marks]
    g = grammar_from_productions(14, prods)
    few = vocab_from_tokens([b"a" + b"".join(b"y" + c for c in w) for w in itertools.product((b"0", b"1", b"2", b"3"), repeat=4)])
    pick = np.random.default_rng(6).integers(0, few.V, size=32_000)
    vocab = _check_repeated(lib, g, few, pick)
    ws = torch.zeros(lib.load_library().cfgzip_displacements_workspace_bytes(vocab.V, g.N, g.P), dtype=torch.uint8, device="cuda")
    lib.cfgzip_displacements(torch.from_numpy(vocab.tok_bytes).cuda(), torch.from_numpy(vocab.tok_off).cuda(), *_grammar_dev(g),
                             g.N, workspace=ws)
    assert int(ws[:8].view(torch.int32)[1]) < 3_200
