"""GPU parity of the class builder's grouping by hash table where it can go wrong: vocabulary sizes
around its workgroups (128 and, above 16,384 tokens, 1,024 tokens each) and mark stretches (256), and class shapes from one class
(every token enters the same entry, with every first byte) to one class per token (tables at their
fullest), from both comparison sources, and with hashes that collide (the sort then takes over)."""

import numpy as np
import pytest

from synthetic_inputs.vocab import vocab_from_tokens
from test_gpu_build import _check_build

pytestmark = pytest.mark.gpu

torch = pytest.importorskip("torch")


@pytest.fixture(scope="module")
def lib():
    import paper_2605_29986_amd as p
    p.load_library()
    return p


def _case(shape, V, seed):
    rng = np.random.default_rng(seed)
    if shape == "one class":  # every byte keeps every state
        S = 24
        table = np.repeat(np.arange(S, dtype=np.uint16)[:, None], 256, axis=1)
        lens = rng.integers(0, 4, size=V)
    elif shape == "last byte":  # 256 small images: many groups of one class
        S = 40
        table = np.tile((np.arange(256) % S).astype(np.uint16), (S, 1))
        lens = rng.integers(0, 5, size=V)
    else:  # "distinct": long tokens over a random automaton
        S = 72
        table = rng.integers(0, S, size=(S, 256)).astype(np.uint16)
        lens = np.full(V, 7)
    toks = [rng.integers(0, 256, size=int(k), dtype=np.uint8).tobytes() for k in lens]
    return vocab_from_tokens(toks), table


@pytest.mark.parametrize("shape", ["one class", "last byte", "distinct"])
@pytest.mark.parametrize("V", [1, 127, 128, 129, 257, 4097, 16_384, 16_385, 20_481])
def test_sizes_and_shapes(lib, V, shape):
    print(f"case V={V} {shape}", flush=True)
    vocab, table = _case(shape, V, V)
    C, coll = _check_build(lib, vocab, table)
    assert coll == 0
    if shape == "one class":
        assert C == 1


@pytest.mark.parametrize("n", [255, 256, 257, 264, 511, 512, 513])
def test_widest_images_that_are_kept(lib, n):
    """Bytes that leave n of 600 states: up to 512 states per token are kept for the comparison, beyond that the
    builder walks again."""
    print(f"case n={n}", flush=True)
    rng = np.random.default_rng(n)
    S = 600
    table = rng.integers(0, S, size=(S, 256)).astype(np.uint16)
    for b in range(8):
        table[:, b] = rng.permutation(S)[:n][np.arange(S) % n]
    toks = [rng.integers(0, 8, size=int(k), dtype=np.uint8).tobytes() for k in rng.integers(0, 4, size=700)]
    _check_build(lib, vocab_from_tokens(toks), table)
    _check_build(lib, vocab_from_tokens(toks), table, stored=False)


@pytest.mark.parametrize("stored", [True, False])
def test_colliding_hashes_are_settled(lib, stored):
    vocab, table = _case("last byte", 1500, 5)
    _, coll = _check_build(lib, vocab, table, stored=stored, hash_override=lambda h: h & 1)
    assert coll > 0
