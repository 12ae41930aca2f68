"""GPU parity of the CSR build (rdf2v_build_csr, through the C ABI) against the oracle on graphs
made to reach the edge cases of its kernels, bit-exact (row_ptr and edges whole):

* row_ptr comes from one pass over the sorted subjects that fills at most 64 entities per
  change of subject (one on sparse graphs), the rest by binary search: runs of 62 to 66 and 127 to 129 entities
  without out-edges between subjects, before the first subject and after the last;
* the digit counts add a wave's equal digits with one atomic: tiles that hold one hub's
  triples only, tiles half hub and half others, and tiles mixing many hubs;
* the radix passes spread the id bits evenly: id spaces of 1 to 31 bits, so every pass count
  and digit width is used, with tile counts below, at and above a multiple of the 8 XCDs."""

import numpy as np
import pytest
import torch

import oracle
import paper_2508_01073_amd as rd
from gpu_helpers import assert_csr_equal, gpu_csr, new_status, say, to_dev

pytestmark = pytest.mark.gpu


def _check(s, p, o, V, P, what):
    s, p, o = (np.asarray(x, dtype=np.int32) for x in (s, p, o))
    rp, ed = oracle.build_csr(s, p, o, V, P)
    csr = gpu_csr(s, p, o, V, P)
    assert_csr_equal(csr, rp, ed)
    say(f"[csr build] {what}: {len(s):,} triples, V={V:,} bit-exact")


@pytest.mark.parametrize("gap", [1, 2, 62, 63, 64, 65, 66, 127, 128, 129, 1000])
def test_runs_of_sinks_between_subjects(gap):
    # subjects every `gap + 1` ids, starting after a gap and leaving one at the end
    rng = np.random.default_rng(gap)
    subjects = np.arange(gap, 40_000, gap + 1)
    V = int(subjects[-1]) + gap + 1
    T = 60_000
    s = rng.choice(subjects, T)
    _check(s, rng.integers(0, 7, T), rng.integers(0, V, T), V, 7, f"subjects every {gap + 1}")


@pytest.mark.parametrize("V", [1, 2, 65, 66, 130, 100_000])
def test_one_subject_at_either_end(V):
    rng = np.random.default_rng(V)
    for subj in sorted({0, V - 1}):
        T = 5_000
        _check(np.full(T, subj), rng.integers(0, 3, T), rng.integers(0, V, T), V, 3, f"only subject {subj}")


def test_hub_only_and_mixed_tiles():
    rng = np.random.default_rng(3)
    V, P = 300_000, 11
    T = 2_000_000
    # 70% of the triples on one hub (whole tiles of it after the first pass), 20% on 40 other
    # hubs, 10% spread: tiles of one key, tiles split between hubs, tiles of many keys
    hubs = rng.choice(V, 41, replace=False)
    kind = rng.random(T)
    s = np.where(kind < 0.7, hubs[0], np.where(kind < 0.9, rng.choice(hubs[1:], T), rng.integers(0, V, T)))
    _check(s, rng.integers(0, P, T), rng.integers(0, V, T), V, P, "hub tiles")


@pytest.mark.parametrize("bits", [1, 2, 7, 8, 9, 13, 16, 17, 18, 19, 24, 26])
@pytest.mark.parametrize("tiles", [1, 7, 8, 9, 23])
def test_id_widths_and_tile_counts(bits, tiles):
    rng = np.random.default_rng(bits * 100 + tiles)
    V = (1 << bits) - rng.integers(0, min(1 << (bits - 1), 5))  # just below a power of two
    T = tiles * 4096 - (0 if tiles % 2 else 1000)               # whole and ragged last tiles
    s = rng.integers(0, V, T)
    s[: T // 10] = V - 1                                        # the largest id, repeated
    _check(s, rng.integers(0, 5, T), rng.integers(0, V, T), int(V), 5, f"{bits}-bit ids, {tiles} tiles")


def test_bad_ids_still_flagged_in_every_column():
    # Subjects are checked by the first count pass, predicates and objects by the first scatter.
    V, P, T = 1000, 4, 20_000
    rng = np.random.default_rng(9)
    base = [rng.integers(0, V, T).astype(np.int32), rng.integers(0, P, T).astype(np.int32),
            rng.integers(0, V, T).astype(np.int32)]
    for col, bad in [(0, V), (0, -1), (1, P), (1, -5), (2, V + 3), (2, -2)]:
        for at in (0, 4095, 4096, T - 1):                        # tile boundaries and the ragged tail
            cols = [c.copy() for c in base]
            cols[col][at] = bad
            st = new_status()
            rd.rdf2v_build_csr(*(to_dev(c) for c in cols), V, P, status=st)
            assert int(st.item()) & rd.RDF2V_STATUS_ID_OUT_OF_RANGE, (col, bad, at)
    st = new_status()
    rd.rdf2v_build_csr(*(to_dev(c) for c in base), V, P, status=st)
    assert int(st.item()) == 0


@pytest.mark.parametrize("T,V", [
    (1, 1), (8192, 16_384), (8191, 16_385), (77, 1 << 24),     # one workgroup, row_ptr inside it or not
    (8193, 1), (8193, 1000), (8193, 16_385),                   # two tiles; keys of 0 and 2 bytes
    (8193, 1 << 26), (12_289, 1 << 26),                        # a table in row_ptr, 4-byte and 2-byte last keys
    (30_001, 1 << 20), (100_003, 262_145),                     # two passes of 9 and 10 bits
    (1 << 21, 100_000), ((1 << 21) + 5, 3), ((1 << 22) + 1, 3_000_000),  # tiles of 2, 4 and 8 rounds
    (1_000_003, (1 << 25) + 1),                                # 9, 7 and 10 bits
])
def test_tile_and_digit_plans(T, V):
    say(f"[csr] plan T={T} V={V}")
    rng = np.random.default_rng(T + V)
    s = rng.integers(0, V, T).astype(np.int32)
    s[rng.random(T) < 0.3] = V - 1                # a hub at the top of the id range
    s[rng.random(T) < 0.2] = V // 3
    p = rng.integers(0, 7, T).astype(np.int32)
    o = rng.integers(0, V, T).astype(np.int32)
    st = new_status()
    csr = rd.rdf2v_build_csr(to_dev(s), to_dev(p), to_dev(o), V, 7, status=st)
    starts = rd.rdf2v_nonsink_starts(csr)
    torch.cuda.synchronize()
    assert int(st.item()) == 0
    order = np.argsort(s, kind="stable")
    assert np.array_equal(csr.edges.cpu().numpy(), np.stack([p[order], o[order]], axis=1))
    degree = np.bincount(s, minlength=V)
    row_ptr = np.zeros(V + 1, np.int64)
    np.cumsum(degree, out=row_ptr[1:])
    assert np.array_equal(csr.row_ptr.cpu().numpy(), row_ptr)
    assert np.array_equal(starts.cpu().numpy(), np.flatnonzero(degree))


@pytest.mark.parametrize("T,V", [(5_000, 1_000), (8_192, 8_000), (9_000, 500), (20_000, 3_000), (60_000, 50_000),
                                 (400_000, 300_000), (1_200_000, 100_000)])
@pytest.mark.parametrize("column", [0, 1, 2])
def test_row_ptr_in_place_of_an_input(T, V, column):
    # row_ptr written over a column of the triples, from its first element and from somewhere inside
    say(f"[csr] row_ptr over column {column}, T={T} V={V}")
    P = 7
    rng = np.random.default_rng(T + V + column)
    s, p, o = (rng.integers(0, n, T).astype(np.int32) for n in (V, P, V))
    rp, ed = oracle.build_csr(s, p, o, V, P)
    for first in (0, (T - V - 1) // 2):
        cols = [to_dev(x) for x in (s, p, o)]
        st = new_status()
        csr = rd.rdf2v_build_csr(*cols, V, P, status=st, row_ptr=cols[column][first:first + V + 1])
        torch.cuda.synchronize()
        assert int(st.item()) == 0
        assert_csr_equal(csr, rp, ed)


@pytest.mark.parametrize("T,V", [(9_000, 35_999), (9_000, 36_000), (20_000, 1_000_000), (8_193, 5_000_000),
                                 ((1 << 19) - 1, 1 << 21), (1 << 19, 1 << 21)])
@pytest.mark.parametrize("clustered", [False, True])
def test_gaps_of_sparse_graphs(T, V, clustered):
    # Four entities per triple or more, below 2^19 triples: a subject writes its own row_ptr entry
    # only and the gap before it is searched. Either side of both limits, with subjects spread over
    # the ids and with a few runs of them (long gaps beside rows without one).
    rng = np.random.default_rng(T + V)
    s = rng.integers(0, V, T)
    if clustered:
        s = (rng.choice([0, 1, V // 2, V - 300], T) + rng.integers(0, 300, T)) % V
    _check(s, rng.integers(0, 7, T), rng.integers(0, V, T), V, 7, f"sparse, clustered={clustered}")
