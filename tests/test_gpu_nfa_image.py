"""GPU parity of the relations' image walk where it can go wrong: numbers of different successor sets around a wave
and around what the walk shares (beyond which every state walks for itself), sets of no, one, two and more members,
row widths that are and are not whole 16-byte units, vocabularies around a workgroup's waves, more first bytes than a
workgroup keeps the sets of, and both sides of the rule that takes a call there (917,504 pairs of token and state, 64
states)."""

import numpy as np
import pytest

from synthetic_inputs.nfa import make_lexer_nfa
from synthetic_inputs.vocab import make_vocab_mixture, vocab_from_tokens
from test_gpu_nfa import _check

pytestmark = pytest.mark.gpu

torch = pytest.importorskip("torch")


@pytest.fixture(scope="module")
def lib():
    import paper_2605_29986_amd as p
    p.load_library()
    return p


def _tokens(rng, V):
    toks = [bytes(rng.integers(0, 7, size=int(n)).astype(np.uint8)) for n in rng.integers(0, 9, size=V)]
    return vocab_from_tokens(toks + [bytes([0, 1, 2, 3, 4, 5] * 30), bytes([0] * 64), bytes([1] * 65), bytes([9, 0])])


@pytest.mark.parametrize("S", [97, 128, 224, 256])
@pytest.mark.parametrize("n", [1, 63, 64, 65, 95, 96, 97])
def test_numbers_of_sets(lib, S, n):
    """On byte k the states fall into n groups, each with a set of 0 to 4 successors.  As many tokens as it takes to come
    to the image walk; with 128 states and more they are one a wave at the most, and a token that every state walks for
    itself is then shared out among the waves."""
    print(f"case S={S} n={n}", flush=True)
    rng = np.random.default_rng(1000 * S + n)
    nfa = np.zeros((256, S, (S + 31) // 32), np.uint32)
    for b in range(6):
        sets = []
        while len(sets) < n:
            s = tuple(sorted(set(int(x) for x in rng.integers(0, S, size=1 + len(sets) % 4)))) if sets else ()
            if s not in sets or not s:  # the empty set may come up again: fewer sets then
                sets.append(s)
        group = np.concatenate([np.arange(n), rng.integers(0, n, size=S - n)])
        rng.shuffle(group)
        for q in range(S):
            for x in sets[group[q]]:
                nfa[b, q, x >> 5] |= np.uint32(1 << (x & 31))
    _check(lib, _tokens(rng, 917_504 // S + 60), nfa)


@pytest.mark.parametrize("V", [1, 15, 16, 17, 4097])
def test_vocabulary_sizes(lib, V):
    _check(lib, make_vocab_mixture(V, V, 40), make_lexer_nfa(5, 200))


@pytest.mark.parametrize("S,V", [(64, 14_400), (65, 14_115), (65, 14_116), (128, 7_168), (128, 7_169), (256, 3_584),
                                 (256, 3_585), (200, 8_192), (200, 8_193), (200, 16_385)])
def test_rule(lib, S, V):
    """Around the number of pairs and of states from which the image walk is taken, and around a token per wave."""
    print(f"case S={S} V={V}", flush=True)
    nfa = make_lexer_nfa(5, max(S, 128))[:, :S, :(S + 31) // 32].copy()
    if S % 32:
        nfa[:, :, -1] &= np.uint32((1 << (S % 32)) - 1)
    rng = np.random.default_rng(S)
    for q in range(S):  # on one byte every state has a set of its own: more of them than are shared
        nfa[ord("9"), q, q >> 5] |= np.uint32(1 << (q & 31))
        x = int(rng.integers(0, S))
        nfa[ord("9"), q, x >> 5] |= np.uint32(1 << (x & 31))
    _check(lib, make_vocab_mixture(V, V, 16), nfa)


@pytest.mark.parametrize("V", [33_000, 50_000])
def test_more_first_bytes_than_are_kept(lib, V):
    """Tokens that begin with every byte alike: a workgroup of 65 or 96 tokens meets more first bytes than the 64 it
    keeps the sets of, and which ones depends on which wave is first."""
    print(f"case V={V}", flush=True)
    rng = np.random.default_rng(V)
    S = 70
    nfa = np.zeros((256, S, 3), np.uint32)
    b, q = np.repeat(np.arange(256), S), np.tile(np.arange(S), 256)
    for _ in range(2):
        x = rng.integers(0, S, size=b.size) % (1 + b % 9)  # a few targets a byte
        np.bitwise_or.at(nfa, (b, q, x >> 5), np.uint32(1) << (x & 31).astype(np.uint32))
    vocab = vocab_from_tokens([rng.integers(0, 256, size=int(k), dtype=np.uint8).tobytes()
                               for k in rng.integers(0, 5, size=V)])
    _check(lib, vocab, nfa)


@pytest.mark.parametrize("V", [4_000, 9_000])
def test_hash_is_optional(lib, V):
    from gpu_util import dev
    nfa = make_lexer_nfa(5, 256)
    nfa[ord("9")] |= np.eye(256, dtype=np.uint32)[:, :8]  # more sets than are shared
    for q in range(256):
        nfa[ord("9"), q, q >> 5] |= np.uint32(1 << (q & 31))
    vocab = make_vocab_mixture(V, V, 16)
    tb, to, nd = dev(vocab.tok_bytes), dev(vocab.tok_off), dev(nfa)
    rel, _ = lib.cfgzip_nfa_signatures(tb, to, nd)
    rel2, h2 = lib.cfgzip_nfa_signatures(tb, to, nd, want_hash=False)
    assert h2 is None and torch.equal(rel, rel2)
