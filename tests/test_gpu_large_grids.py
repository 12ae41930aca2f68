"""Calls whose kernels need 2^32 threads or more, which one HIP launch does not run: walks without a
hop, duplicate-free walks in long groups, skip-gram pairs and CBOW examples of so many walk rows, nearly
all of them empty, and vocabularies with large bounds. The rows with tokens lie at the ends and around
the place where the launches are cut; outputs are compared whole (tolerance 0)."""

import numpy as np
import pytest
import torch

import oracle
import paper_2508_01073_amd as rd
from gpu_helpers import device, new_status, say, to_dev

pytestmark = [pytest.mark.gpu, pytest.mark.slow]


def _rows(n, width, cut, seed):
    """n rows on the device, empty but for some at both ends and around row `cut`; and those rows."""
    rng = np.random.default_rng(seed)
    at = np.unique(np.concatenate([np.arange(40), cut + np.arange(-40, 40), n - 1 - np.arange(5), rng.integers(0, n, 500)]))
    at = at[at < n]
    ln = rng.integers(0, width + 1, len(at)).astype(np.int32)
    tok = np.where(np.arange(width) < ln[:, None], rng.integers(0, 10**6, (len(at), width)), -1).astype(np.int32)
    tokens = torch.zeros((n, width), dtype=torch.int32, device=device())
    lens = torch.zeros(n, dtype=torch.int32, device=device())
    where = torch.from_numpy(at).to(device())
    tokens[where] = to_dev(tok)
    lens[where] = to_dev(ln)
    return tokens, lens, tok, ln


def test_pairs_of_more_rows_than_one_launch():
    # 33 tokens, window 16: a walk per 64-thread block
    n, width, window = (1 << 26) + 5, 33, 16
    say(f"[large grids] pairs of {n:,} rows of {width}")
    tokens, lens, tok, ln = _rows(n, width, (1 << 26) - 1024, 1)
    st = new_status()
    pairs = rd.rdf2v_skipgram_pairs(tokens, lens, window, status=st)
    assert int(st.item()) == 0
    assert np.array_equal(pairs.cpu().numpy(), oracle.skipgram_pairs(tok, ln, window))


def test_cbow_of_more_rows_than_one_launch():
    # 33 tokens, window 8: three walks per 128-thread block
    n, width, window = 3 * (1 << 25) + 7, 33, 8
    say(f"[large grids] CBOW examples of {n:,} rows of {width}")
    tokens, lens, tok, ln = _rows(n, width, 3 * ((1 << 25) - 1024), 2)
    st = new_status()
    centers, contexts = rd.rdf2v_cbow_examples(tokens, lens, window, status=st)
    assert int(st.item()) == 0
    ref_c, ref_x = oracle.cbow_examples(tok, ln, window)
    assert np.array_equal(centers.cpu().numpy(), ref_c) and np.array_equal(contexts.cpu().numpy(), ref_x)


def test_walks_of_more_rows_than_one_launch():
    wpn = (1 << 30) + 64
    n = 4 * wpn + wpn // 1000
    say(f"[large grids] {n:,} walks of no hop")
    csr = rd.rdf2v_build_csr(to_dev([0, 1, 2]), to_dev([0, 0, 0]), to_dev([1, 2, 0]), 7, 1)
    starts = [3, 0, 6, 2, 5]
    tokens = torch.full((n, 1), -7, dtype=torch.int32, device=device())
    lens = torch.full((n,), -7, dtype=torch.int32, device=device())
    st = new_status()
    rd.rdf2v_random_walks(csr, to_dev(starts), wpn, 0, 1, 0, n, tokens=tokens, lens=lens, status=st)
    assert int(st.item()) == 0
    for i, v in enumerate(starts):
        rows = slice(i * wpn, min(n, (i + 1) * wpn))
        assert bool((tokens[rows] == v).all()) and bool((lens[rows] == 1).all())


def test_long_groups_of_more_rows_than_one_launch():
    # groups of 2,000 rows of no token: the first of each is kept, and the rows of one token
    n, group = (1 << 32) + 3_000, 2_000
    say(f"[large grids] duplicate-free walks of {n:,} rows in groups of {group}")
    rng = np.random.default_rng(4)
    named = np.concatenate([[1], (1 << 32) + np.arange(-6, 6), [n - 1], rng.integers(0, n, 200)])
    named = np.unique(named[named % group != 0])
    named = named[np.concatenate([[True], named[1:] // group != named[:-1] // group])]  # one to a group
    where = torch.from_numpy(named).to(device())
    tokens = torch.zeros((n, 1), dtype=torch.int32, device=device())
    lens = torch.zeros(n, dtype=torch.int32, device=device())
    tokens[where] = 5
    lens[where] = 1
    st = new_status()
    tok, ln = rd.rdf2v_unique_walks(tokens, lens, group, status=st)
    assert int(st.item()) == 0
    kept = np.union1d(np.arange(0, n, group), named)
    is_named = np.isin(kept, named)
    assert np.array_equal(ln.cpu().numpy(), is_named.astype(np.int32))
    assert np.array_equal(tok.cpu().numpy()[:, 0], np.where(is_named, 5, 0))


@pytest.mark.parametrize("max_entities,max_predicates", [
    (1 << 27, 1 << 27),  # two tables of 2^28 slots, reset by 2^32 threads together
    (1 << 28, 1000),     # one of 2^29
])
def test_vocabulary_with_large_bounds(max_entities, max_predicates):
    n = (1 << 26) + 100
    say(f"[large grids] vocabulary of {n:,} triples, bounds {max_entities:,} and {max_predicates:,}")
    rng = np.random.default_rng(3)
    junk = torch.full((1 << 34,), 0x5A, dtype=torch.uint8, device=device())  # the tables are not zeroed memory
    del junk
    cols, keys = [], []
    for c in range(3):
        at = np.unique(np.concatenate([np.arange(20), rng.integers(0, n, 300), [n - 1]]))
        key = rng.integers(0, 200, len(at))  # three decimal digits; every other string is empty
        size = torch.zeros(n, dtype=torch.int64, device=device())
        size[torch.from_numpy(at).to(device())] = 3
        off = torch.zeros(n + 1, dtype=torch.int64, device=device())
        torch.cumsum(size, 0, out=off[1:])
        chars = np.frombuffer("".join(f"{k:03d}" for k in key).encode(), np.uint8).copy()
        cols.append((torch.from_numpy(chars).to(device()), off))
        ids = np.zeros(n, np.int16)  # 0: the empty string, else 1 + the key
        ids[at] = 1 + key
        keys.append(ids)
    st = new_status()
    s, p, o, counts = rd.rdf2v_build_vocabulary(cols[0], cols[1], cols[2], max_entities, max_predicates, status=st)
    assert int(st.item()) == 0

    def by_first_appearance(seq):
        named = np.flatnonzero(seq)
        values, first = np.unique(seq[named], return_index=True)
        order = np.argsort(np.concatenate([[np.argmin(seq)], named[first]]))  # of the empty string and the keys
        rank = np.zeros(int(seq.max()) + 1, np.int32)
        rank[np.concatenate([[0], values])[order]] = np.arange(len(order))
        return rank[seq], len(order)

    ent, n_ent = by_first_appearance(np.stack([keys[0], keys[2]], axis=1).reshape(-1))
    pred, n_pred = by_first_appearance(keys[1])
    assert counts.cpu().tolist() == [n_ent, n_pred]
    assert np.array_equal(s.cpu().numpy(), ent[0::2]) and np.array_equal(o.cpu().numpy(), ent[1::2])
    assert np.array_equal(p.cpu().numpy(), pred)
