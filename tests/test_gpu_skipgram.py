"""GPU parity for skip-gram pair generation (through the C ABI) against the
oracle, bit-exact: small rows of every length, real walk rows at several
windows, capacity truncation, and slices of the full power-law corpus."""

import numpy as np
import pytest
import torch

import oracle
import paper_2508_01073_amd as rd
import synth
from gpu_helpers import device, gpu_csr, gpu_walks, new_status, say, to_dev

pytestmark = pytest.mark.gpu


def _gpu_pairs(tok, ln, window):
    st = new_status()
    pairs = rd.rdf2v_skipgram_pairs(tok, ln, window, status=st)
    torch.cuda.synchronize()
    rd.check_device_status(st, "rdf2v_skipgram_pairs")
    return pairs.cpu().numpy()


@pytest.mark.parametrize("width", [1, 2, 9, 17, 33, 129])
@pytest.mark.parametrize("window", [0, 1, 2, 5, 64])
def test_random_rows(width, window):
    say(f"[pairs] random rows width={width} window={window}")
    rng = np.random.default_rng(width * 100 + window)
    n = 3000
    ln = rng.integers(0, width + 1, n).astype(np.int32)
    tok = np.full((n, width), -1, np.int32)
    for r in range(n):
        tok[r, :ln[r]] = rng.integers(0, 10**6, ln[r])
    got = _gpu_pairs(to_dev(tok), to_dev(ln), window)
    ref = oracle.skipgram_pairs(tok, ln, window)
    assert got.shape == ref.shape and np.array_equal(got, ref)


@pytest.mark.parametrize("window", [1, 5, 10])
def test_walk_rows_tiny_uniform(window):
    w = synth.WORKLOADS["tiny_uniform"]
    say(f"[pairs] tiny_uniform walks window={window}")
    s, p, o = synth.triples(w)
    csr = gpu_csr(s, p, o, w.num_entities, w.num_predicates, walk_records=True)
    starts = rd.rdf2v_nonsink_starts(csr)
    tok, ln = gpu_walks(csr, starts, w.walks_per_node, w.depth, synth.WALK_SEED)
    got = _gpu_pairs(tok, ln, window)
    ref = oracle.skipgram_pairs(tok.cpu().numpy(), ln.cpu().numpy(), window)
    assert np.array_equal(got, ref)


def test_capacity_and_count():
    say("[pairs] capacity truncation")
    tok = to_dev(np.arange(40, dtype=np.int32).reshape(4, 10))
    ln = to_dev(np.array([10, 3, 0, 7], np.int32))
    ref = oracle.skipgram_pairs(tok.cpu().numpy(), ln.cpu().numpy(), 3)
    out = torch.full((20, 2), -5, dtype=torch.int32, device=device())
    st = new_status()
    pairs, count = rd.rdf2v_skipgram_pairs(tok, ln, 3, pairs=out, status=st)
    torch.cuda.synchronize()
    assert int(count.item()) == ref.shape[0]
    assert np.array_equal(out.cpu().numpy(), ref[:20])
    assert int(st.item()) & rd.RDF2V_STATUS_CAPACITY


def test_bad_lengths_are_flagged():
    say("[pairs] lengths outside the row")
    tok = to_dev(np.zeros((3, 5), np.int32))
    st = new_status()
    rd.rdf2v_skipgram_pairs(tok, to_dev(np.array([2, 9, -1], np.int32)), 2, status=st)
    torch.cuda.synchronize()
    assert int(st.item()) & rd.RDF2V_STATUS_BAD_LENGTH


def test_powerlaw_corpus_slices():
    w = synth.WORKLOADS["powerlaw_20m"]
    say(f"[pairs] {w.describe()}; window 5 over slices of the corpus")
    s, p, o = synth.triples(w)
    csr = gpu_csr(s, p, o, w.num_entities, w.num_predicates, walk_records=True)
    starts = rd.rdf2v_nonsink_starts(csr)
    tok, ln = gpu_walks(csr, starts, w.walks_per_node, w.depth, synth.WALK_SEED)
    n = tok.shape[0]
    # the count over the whole corpus (count-only call) equals the closed form summed over lengths
    count = torch.empty(1, dtype=torch.int64, device=device())
    rd.rdf2v_skipgram_pairs(tok, ln, 5, pairs=torch.empty((0, 2), dtype=torch.int32, device=device()),
                            count=count)
    L = ln.to(torch.int64)
    m = torch.clamp(L - 1, max=5)
    closed = int((2 * (m * L - m * (m + 1) // 2)).clamp(min=0).sum().item())
    assert int(count.item()) == closed
    for b in (0, n // 2, n - 150_000):
        sl_t, sl_l = tok[b:b + 150_000].contiguous(), ln[b:b + 150_000].contiguous()
        got = _gpu_pairs(sl_t, sl_l, 5)
        ref = oracle.skipgram_pairs(sl_t.cpu().numpy(), sl_l.cpu().numpy(), 5)
        assert np.array_equal(got, ref), f"slice at {b}"


@pytest.mark.parametrize("n,width,window,offset", [
    (1, 17, 5, 3), (7, 17, 5, 1), (8, 17, 5, 15),     # one block of 7 walks, its end, the next one
    (28 * 1024, 9, 5, 7), (28 * 1024 + 1, 9, 5, 9),   # one and two workgroups of the count
    (7 * 2048 + 3, 17, 5, 5), (40_000, 3, 2, 11),     # several; blocks of more walks than a wave
    (1500, 100, 64, 2), (2100, 129, 128, 1),          # no stage; a walk per block
])
def test_outputs_at_any_offset_and_cut(n, width, window, offset):
    # Outputs that begin anywhere in a 128-byte line, with room for everything
    # and with room for two thirds: what lies around them is left alone.
    say(f"[pairs] n={n} width={width} window={window} offset={offset}")
    rng = np.random.default_rng(n + width)
    ln = rng.integers(0, width + 1, n).astype(np.int32)
    ln[rng.random(n) < 0.5] = width
    tok = np.where(np.arange(width) < ln[:, None], rng.integers(0, 10**6, (n, width)), -1).astype(np.int32)
    t, l = to_dev(tok), to_dev(ln)
    pairs = oracle.skipgram_pairs(tok, ln, window)
    centers, contexts = oracle.cbow_examples(tok, ln, max(window, 1))
    for part in (1.0, 2 / 3):
        cap = int(len(pairs) * part)
        buf = torch.full((cap + offset + 40, 2), -7, dtype=torch.int32, device=device())
        st = new_status()
        _, cnt = rd.rdf2v_skipgram_pairs(t, l, window, pairs=buf[offset:offset + cap], status=st)
        got = buf.cpu().numpy()
        assert int(cnt.item()) == len(pairs)
        assert np.array_equal(got[offset:offset + cap], pairs[:cap])
        assert (got[:offset] == -7).all() and (got[offset + cap:] == -7).all()
        assert int(st.item()) == (rd.RDF2V_STATUS_CAPACITY if cap < len(pairs) else 0)
        cap = int(len(centers) * part)
        ctr = torch.full((cap + offset + 40,), -7, dtype=torch.int32, device=device())
        ctx = torch.full(((cap + 40) * 2 * max(window, 1) + offset,), -7, dtype=torch.int32, device=device())
        wide = 2 * max(window, 1) * cap
        st = new_status()
        _, _, cnt = rd.rdf2v_cbow_examples(t, l, max(window, 1), centers=ctr[offset:offset + cap],
                                           contexts=ctx[offset:offset + wide], status=st)
        c, x = ctr.cpu().numpy(), ctx.cpu().numpy()
        assert int(cnt.item()) == len(centers)
        assert np.array_equal(c[offset:offset + cap], centers[:cap])
        assert np.array_equal(x[offset:offset + wide], contexts[:cap].reshape(-1))
        assert (c[:offset] == -7).all() and (c[offset + cap:] == -7).all()
        assert (x[:offset] == -7).all() and (x[offset + wide:] == -7).all()
        assert int(st.item()) == (rd.RDF2V_STATUS_CAPACITY if cap < len(centers) else 0)


@pytest.mark.parametrize("width,walks", [(1, 256), (2, 128), (3, 85)])
@pytest.mark.parametrize("blocks", [127, 128, 129, 1025])
def test_narrow_rows_in_many_blocks(width, walks, blocks):
    # more walks to an emit block than a wave has lanes: eight threads count a block, 128 blocks a
    # workgroup; numbers of blocks around one workgroup and several
    for n in (walks * blocks, walks * blocks - 1, walks * (blocks - 1) + 1):
        say(f"[pairs] narrow rows width={width} n={n}")
        rng = np.random.default_rng(n + width)
        ln = rng.integers(0, width + 1, n).astype(np.int32)
        tok = np.where(np.arange(width) < ln[:, None], rng.integers(0, 10**6, (n, width)), -1).astype(np.int32)
        t, l = to_dev(tok), to_dev(ln)
        assert np.array_equal(_gpu_pairs(t, l, 2), oracle.skipgram_pairs(tok, ln, 2))
        centers, contexts = rd.rdf2v_cbow_examples(t, l, 2)
        ref_c, ref_x = oracle.cbow_examples(tok, ln, 2)
        assert np.array_equal(centers.cpu().numpy(), ref_c) and np.array_equal(contexts.cpu().numpy(), ref_x)
