"""GPU parity of drafting where a match occurs at many places: numbers of places and of distinct continuations at the edges
of what one wave, four, eight and sixteen waves take, and of the list in memory.  Whole numbers: everything is compared."""
import numpy as np
import pytest

from test_gpu_draft import _compare, _from_lists

pytestmark = pytest.mark.gpu


@pytest.mark.parametrize("places,distinct,gamma,top_k,conf", [
    (1, 1, 8, 4, 0.0), (64, 64, 8, 4, 0.0), (65, 65, 8, 1, 0.0), (256, 7, 8, 4, 0.1), (511, 300, 3, 16, 0.0), (512, 512, 8, 3, 0.0),
    (513, 40, 8, 4, 0.0), (513, 513, 10, 2, 0.0), (700, 65, 3, 2, 0.0), (1024, 1000, 8, 4, 0.002), (1025, 513, 5, 2, 0.0),
    (2048, 2048, 8, 4, 0.0), (2048, 1, 8, 4, 0.5), (2049, 2048, 8, 4, 0.0), (2049, 64, 8, 1, 0.0), (3000, 2049, 8, 2, 0.0),
    (5000, 3, 8, 4, 0.0), (5000, 600, 9, 3, 0.0), (5000, 600, 8, 3, 0.03), (2100, 50, 2, 4, 0.0), (1500, 900, 20, 3, 0.0)])
def test_a_match_at_many_places(places, distinct, gamma, top_k, conf):
    rng = np.random.default_rng(places * 7 + distinct)
    vocab = 60000
    # continuations that share beginnings of any length: a random tree of tokens, the last ones all different
    strings = np.zeros((distinct, gamma), np.int64)
    for i in range(distinct):
        if i:
            strings[i] = strings[rng.integers(0, i)]
        at = 0 if i == 0 else int(rng.integers(0, gamma))
        strings[i, at:] = rng.integers(0, [3, 40, 50000][int(rng.integers(0, 3))], size=gamma - at)
    strings[:, -1] = np.arange(distinct) if distinct > 1 else 5
    share = np.concatenate([np.arange(min(distinct, places)), rng.integers(0, distinct, size=max(places - distinct, 0))])
    body = [np.concatenate([[vocab - 1, vocab - 2], strings[j]]) for j in rng.permutation(share)]
    seqs = [np.concatenate(body[k::3]).tolist() for k in range(3) if len(body[k::3])]
    # one sequence ends inside a continuation, one with the match itself
    seqs += [[vocab - 1, vocab - 2] + strings[0, :max(gamma // 2, 1)].tolist(), [vocab - 1, vocab - 2]]
    d = _from_lists([seqs], [0, 0], [[vocab - 1, vocab - 2], [vocab - 2]], gamma_max=gamma, top_k=top_k, p_min=1, p_max=4, vocab=vocab,
                    min_confidence=conf)
    d.max_spec_tokens[1] = max(gamma - 1, 1)
    want = _compare(d, "%d places, %d continuations" % (places, distinct))
    assert want[3][0, 0] >= places


@pytest.mark.parametrize("places,others,gamma,top_k,conf", [
    (32767, 1, 8, 4, 0.0), (32768, 1, 8, 1, 0.0), (32768, 2, 8, 4, 0.0), (40000, 3, 5, 12, 0.01), (65535, 1, 3, 1, 0.5), (65535, 2, 8, 4, 0.0),
    (65535, 2, 3, 1, 0.0), (65536, 1, 8, 4, 0.0), (65536, 2, 3, 1, 0.0), (70000, 2, 8, 4, 0.0), (2800, 30, 8, 4, 0.0)])
def test_numbers_of_places_that_need_all_their_sixteen_bits(places, others, gamma, top_k, conf):
    """One token before every place; the tokens behind it are drawn from it and `others` - 1 more, so that one string recurs that often (others = 1) or
    hundreds recur hundreds of times and add up in a level's pairs.  From 65536 places on, the list in memory."""
    rng = np.random.default_rng(places + others)
    s = np.full(places + 1, 7)
    if others > 1:
        s = rng.choice([7] + list(range(100, 99 + others)), size=2 * others * places)
        s = np.concatenate([s[: np.flatnonzero(s == 7)[places - 1] + 1], [100, 100, 100]])
    d = _from_lists([[s.tolist()]], [0], [[7]], gamma_max=gamma, top_k=top_k, p_min=1, p_max=1, vocab=60000, min_confidence=conf)
    want = _compare(d, "%d places of %d tokens" % (places, others))
    assert want[3][0, 0] == places


@pytest.mark.parametrize("n", [0, 1, 64, 65, 130, 512, 513, 1500, 2048, 2049, 4000])
@pytest.mark.parametrize("tail", [0, 1, 5])
@pytest.mark.parametrize("gamma,top_k", [(8, 4), (3, 1), (12, 2), (1, 8), (2, 3)])
def test_one_string_that_most_places_show_beside_ends_and_others(n, tail, gamma, top_k):
    """A phrase of period seven over sequences that end anywhere in it, with sequences of other tokens between: most places of a wave, or
    of all waves, show one string; `n` places or none, `tail` sequences that differ."""
    rng = np.random.default_rng(n + 31 * tail + gamma)
    phrase = list(range(50, 57))
    seqs, left = [], n
    while left > 0:
        k = min(left, int(rng.integers(1, 400)))
        seqs.append(([phrase[i % 7] for i in range(7 * k)] + phrase[: int(rng.integers(1, 8))]))
        left -= k
    for i in range(tail):
        seqs.insert(int(rng.integers(0, len(seqs) + 1)), phrase + rng.integers(100, 130, size=20).tolist())
    seqs.append([900, 901])
    if len(seqs) > 120:
        seqs = seqs[:119] + [sum(seqs[119:], [])]
    d = _from_lists([seqs], [0, 0], [phrase[5:] if n else [333], phrase[:3]], gamma_max=gamma, top_k=top_k, p_min=2, p_max=4, vocab=60000)
    _compare(d, "%d places, %d others" % (n, tail))
