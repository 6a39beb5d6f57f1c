"""GPU parity of the relations' image walk where it can go wrong: numbers of different successor sets around a wave
and around what the walk shares (beyond which every state walks for itself), sets of no, one, two and more members,
row widths that are and are not whole 16-byte units, and vocabularies around a workgroup's waves."""

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
    """On byte k the states fall into n groups, each with a set of 0 to 4 successors."""
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
    _check(lib, _tokens(rng, 300), nfa)


@pytest.mark.parametrize("V", [1, 15, 16, 17, 4097])
def test_vocabulary_sizes(lib, V):
    _check(lib, make_vocab_mixture(V, V, 40), make_lexer_nfa(5, 200))
