"""GPU parity for BFS walks (through the C ABI) against the oracle, bit-exact:
hand-built graphs, random multigraphs and generated workloads, with depth
limits, truncation at max_walks, sink and repeated roots."""

import numpy as np
import pytest
import torch

import oracle
import paper_2508_01073_amd as rd
import synth
from gpu_helpers import device, gpu_csr, new_status, say, to_dev

pytestmark = pytest.mark.gpu


def _compare(csr, rp, ed, V, P, roots, depth, max_walks, what, expect_capacity=None):
    st = new_status()
    tok, ln, cnt = rd.rdf2v_bfs_walks(csr, to_dev(roots), depth, max_walks, status=st)
    torch.cuda.synchronize()
    flags = int(st.item())
    ref_t, ref_l, ref_c, trunc = oracle.bfs_walks(rp, ed, V, P, roots, depth, max_walks)
    cnt = cnt.cpu().numpy()
    assert np.array_equal(cnt, ref_c), f"{what}: walk counts differ"
    tok = tok.cpu().numpy()
    ln = ln.cpu().numpy()
    for r in range(len(roots)):
        k = ref_c[r]
        if not (np.array_equal(tok[r, :k], ref_t[r, :k]) and np.array_equal(ln[r, :k], ref_l[r, :k])):
            raise AssertionError(f"{what}: root {roots[r]} differs: gpu {tok[r, :k].tolist()[:3]} "
                                 f"oracle {ref_t[r, :k].tolist()[:3]}")
    assert bool(flags & rd.RDF2V_STATUS_CAPACITY) == (trunc > 0), what
    assert not flags & ~rd.RDF2V_STATUS_CAPACITY, f"{what}: status {flags}"
    return ref_c


def test_hand_graphs():
    say("[bfs] hand graphs")
    tr = [(0, 0, 1), (0, 1, 2), (1, 0, 3), (2, 1, 3), (3, 0, 0)]
    t = np.array(tr, np.int32)
    rp, ed = oracle.build_csr(t[:, 0], t[:, 1], t[:, 2], 4, 2)
    csr = gpu_csr(t[:, 0], t[:, 1], t[:, 2], 4, 2)
    for depth in (0, 1, 2, 3, 5):
        _compare(csr, rp, ed, 4, 2, np.array([0, 3, 2, 1, 0], np.int32), depth, 5, f"diamond depth {depth}")
    star = np.array([(0, j % 2, j) for j in range(1, 12)] + [(5, 1, 0)], np.int32)
    rp, ed = oracle.build_csr(star[:, 0], star[:, 1], star[:, 2], 12, 2)
    csr = gpu_csr(star[:, 0], star[:, 1], star[:, 2], 12, 2)
    _compare(csr, rp, ed, 12, 2, np.array([0, 7, 5], np.int32), 3, 4, "star truncated")
    _compare(csr, rp, ed, 12, 2, np.array([0, 7, 5], np.int32), 3, 50, "star")


@pytest.mark.parametrize("V,T,depth,seed", [(50, 150, 3, 0), (300, 1200, 4, 1), (2000, 6000, 6, 2),
                                            (5000, 60_000, 2, 3), (40, 30, 10, 4), (5000, 40_000, 3, 5)])
def test_random_multigraphs(V, T, depth, seed):
    say(f"[bfs] random multigraph V={V} T={T} depth={depth}")
    P = 7
    rng = np.random.default_rng(seed)
    s = rng.integers(0, V, T).astype(np.int32)
    p = rng.integers(0, P, T).astype(np.int32)
    o = rng.integers(0, V, T).astype(np.int32)
    s[:5] = 0; o[:2] = 0                        # self-loops and repeated edges at entity 0
    rp, ed = oracle.build_csr(s, p, o, V, P)
    csr = gpu_csr(s, p, o, V, P)
    roots = np.concatenate([np.arange(min(V, 600), dtype=np.int32), np.array([0, 0, V - 1], np.int32)])
    _compare(csr, rp, ed, V, P, roots, depth, V, f"V={V} full")
    _compare(csr, rp, ed, V, P, roots, depth, 7, f"V={V} truncated")


def test_big_levels_and_trees():
    # mean out-degree 20: levels of hundreds and thousands of entities and trees
    # of up to ~20k, past the part of the tree and of a level that is kept in LDS
    say("[bfs] V=20000 T=400000 depth 4, big levels and trees")
    V, P, T = 20_000, 5, 400_000
    rng = np.random.default_rng(11)
    s = rng.integers(0, V, T).astype(np.int32)
    p = rng.integers(0, P, T).astype(np.int32)
    o = rng.integers(0, V, T).astype(np.int32)
    rp, ed = oracle.build_csr(s, p, o, V, P)
    csr = gpu_csr(s, p, o, V, P)
    roots = rng.integers(0, V, 24).astype(np.int32)
    counts = _compare(csr, rp, ed, V, P, roots, 4, V, "big levels")
    assert counts.max() > 5000
    _compare(csr, rp, ed, V, P, roots, 3, 1500, "big levels truncated")


def test_tiny_uniform_all_roots():
    w = synth.WORKLOADS["tiny_uniform"]
    say("[bfs] tiny_uniform, every entity as root, depth 3")
    s, p, o = synth.triples(w)
    V, P = w.num_entities, w.num_predicates
    rp, ed = oracle.build_csr(s, p, o, V, P)
    csr = gpu_csr(s, p, o, V, P)
    counts = _compare(csr, rp, ed, V, P, np.arange(V, dtype=np.int32), 3, 1000, "tiny_uniform")
    assert counts.max() > 100


def test_powerlaw_roots_with_hubs():
    say("[bfs] power law 200k entities, depth 2, hub roots")
    V, P = 200_000, 20
    s, p, o = synth.powerlaw_triples(V, P, 2_000_000, sink_fraction=0.1)
    rp, ed = oracle.build_csr(s, p, o, V, P)
    csr = gpu_csr(s, p, o, V, P)
    deg = np.diff(rp)
    hubs = np.argsort(-deg)[:8].astype(np.int32)
    rng = np.random.default_rng(0)
    roots = np.concatenate([hubs, rng.integers(0, V, 300).astype(np.int32)])
    _compare(csr, rp, ed, V, P, roots, 2, 256, "power law hubs")


def test_out_of_range_root_is_flagged():
    say("[bfs] root out of range")
    t = np.array([(0, 0, 1), (1, 0, 2)], np.int32)
    csr = gpu_csr(t[:, 0], t[:, 1], t[:, 2], 3, 1)
    st = new_status()
    tok, ln, cnt = rd.rdf2v_bfs_walks(csr, to_dev([0, 9, 1]), 2, 4, status=st)
    torch.cuda.synchronize()
    assert int(st.item()) & rd.RDF2V_STATUS_ID_OUT_OF_RANGE
    assert cnt.cpu().tolist() == [1, 0, 1]


@pytest.mark.parametrize("depth,max_walks", [(2, 256), (3, 1024), (3, 40)])
def test_uniform_1m_every_start_sampled(depth, max_walks):
    # the benchmark's launch: every start entity of the 1M-triple uniform graph
    # in one call, trees of ~10^depth entities (up to ~2900 at depth 3); rows of
    # 3000 sampled roots checked against the oracle
    w = synth.WORKLOADS["uniform_1m"]
    say(f"[bfs] uniform_1m every start, depth {depth}, max_walks {max_walks}")
    s, p, o = synth.triples(w)
    V, P = w.num_entities, w.num_predicates
    rp, ed = oracle.build_csr(s, p, o, V, P)
    csr = gpu_csr(s, p, o, V, P)
    roots = oracle.nonsink_starts(rp, V)
    st = new_status()
    tok, ln, cnt = rd.rdf2v_bfs_walks(csr, to_dev(roots), depth, max_walks, status=st)
    torch.cuda.synchronize()
    pick = np.sort(np.random.default_rng(depth * 7 + max_walks).choice(len(roots), 3000, replace=False))
    ref_t, ref_l, ref_c, trunc = oracle.bfs_walks(rp, ed, V, P, roots[pick], depth, max_walks)
    cnt = cnt.cpu().numpy()
    assert np.array_equal(cnt[pick], ref_c)
    tok = tok[torch.from_numpy(pick).to(device())].cpu().numpy()
    ln = ln[torch.from_numpy(pick).to(device())].cpu().numpy()
    for i in range(len(pick)):
        k = ref_c[i]
        assert np.array_equal(tok[i, :k], ref_t[i, :k]) and np.array_equal(ln[i, :k], ref_l[i, :k]), roots[pick[i]]
    flags = int(st.item())
    assert not flags & ~rd.RDF2V_STATUS_CAPACITY
    if trunc > 0:
        assert flags & rd.RDF2V_STATUS_CAPACITY
    if flags & rd.RDF2V_STATUS_CAPACITY:
        assert (cnt == max_walks).any()


def test_trees_around_storage_limits():
    # Roots whose trees have about 500 or 1000 entities above the depth limit,
    # or about 1500 or 3000 in all: on both sides of the sizes where the kernels
    # hand a root from the small on-chip tier to the big one and from there to
    # the workspace pass; children reached twice, back edges into the tree and
    # shuffled entity ids.
    say("[bfs] trees around the on-chip storage limits")
    V, P = 40_000, 3
    rng = np.random.default_rng(5)
    ids = rng.permutation(V).astype(np.int64)
    nxt = [0]

    def fresh(n):
        out = ids[nxt[0]:nxt[0] + n]
        nxt[0] += n
        return out

    trip = []
    roots = []

    def fan(root, kids, grand_per_kid):
        for c in kids:
            trip.append((root, int(rng.integers(P)), c))
        trip.append((root, 0, kids[0]))                 # reached twice
        for c in kids:
            for g in fresh(grand_per_kid):
                trip.append((c, int(rng.integers(P)), g))
            if grand_per_kid:
                trip.append((c, 1, root))               # back edge into the tree

    for n_kids in (510, 511, 512, 1022, 1023, 1024, 1534, 1535, 1536, 3071, 3072):
        r = fresh(1)[0]
        roots.append(r)
        fan(r, fresh(n_kids), 0)
    for n_grand in (1533, 1534, 1535, 3069, 3070, 3071):
        r = fresh(1)[0]
        roots.append(r)
        fan(r, fresh(1), n_grand)
    r = fresh(1)[0]
    roots.append(r)
    fan(r, fresh(40), 75)                               # 1 + 40 + 3000 entities
    t = np.array(trip, np.int64)
    rng.shuffle(t)
    s, p, o = (t[:, k].astype(np.int32) for k in range(3))
    rp, ed = oracle.build_csr(s, p, o, V, P)
    csr = gpu_csr(s, p, o, V, P)
    roots = np.array(roots + roots[:3], np.int32)
    for depth in (1, 2, 3):
        _compare(csr, rp, ed, V, P, roots, depth, 4000, f"limits depth {depth}")
        _compare(csr, rp, ed, V, P, roots, depth, 1500, f"limits depth {depth} truncated")


def test_inconsistent_csr_is_flagged_not_read():
    # row_ptr decreasing at entity 1, past num_edges at entity 2 and 3: every row
    # is checked before its records are read, so BFS only raises the status bit
    say("[bfs] inconsistent CSR")
    dev = device()
    row_ptr = torch.tensor([0, 3, 1, 50, 4], dtype=torch.int32, device=dev)
    edges = torch.tensor([[0, 1], [0, 2], [0, 1], [0, 3]], dtype=torch.int32, device=dev)
    csr = rd.Csr(row_ptr, edges, 4, 1)
    for roots in ([0], [1], [2, 3], [0, 1, 2, 3] * 50):
        st = new_status()
        tok, ln, cnt = rd.rdf2v_bfs_walks(csr, to_dev(roots), 3, 8, status=st)
        torch.cuda.synchronize()
        assert int(st.item()) & rd.RDF2V_STATUS_BAD_CSR, roots
        assert bool((cnt >= 0).all()) and bool((cnt <= 8).all())


@pytest.mark.parametrize("V,fan,depth,max_walks", [
    (30_000, 9_000, 2, 64),          # a row long enough to be streamed once the walks are known
    (30_000, 9_000, 3, 40_000),      # every walk kept: levels of many row windows, in order
    (1_000_000, 60_000, 2, 300),     # the largest bitmaps that fit LDS
    (1_300_000, 60_000, 3, 300),     # bitmap in the workspace
    (1_300_000, 420_000, 2, 300),    # more tree nodes than a slice of 512 holds: rerun with larger slices
])
def test_trees_beyond_the_lds_tiers(V, fan, depth, max_walks):
    say(f"[bfs] hub trees V={V} fan={fan} depth={depth}")
    P = 9
    rng = np.random.default_rng(V + fan + depth)
    ids = rng.permutation(V).astype(np.int32)
    root, hub, rest = ids[0], ids[1], ids[2:]
    hub_row = rng.choice(rest, 3 * fan if 3 * fan < V else fan).astype(np.int32)  # with repeats
    n_more = min(V, 50_000)
    s = np.concatenate([np.full(fan, root), np.full(len(hub_row), hub), rng.choice(rest[:fan], n_more)])
    o = np.concatenate([rest[:fan], hub_row, rng.choice(ids, n_more)])
    s = np.concatenate([s, rest[:3], rest[fan // 2:fan // 2 + 2]]).astype(np.int32)  # ways into the hub
    o = np.concatenate([o, np.full(5, hub)]).astype(np.int32)
    order = rng.permutation(len(s))
    s, o = s[order], o[order]
    p = rng.integers(0, P, len(s)).astype(np.int32)
    rp, ed = oracle.build_csr(s, p, o, V, P)
    csr = gpu_csr(s, p, o, V, P)
    many = rest[-560:] if max_walks < 1000 else rest[-20:]
    roots = np.concatenate([[root, hub, rest[0], root], many, rest[fan // 2:fan // 2 + 1]]).astype(np.int32)
    counts = _compare(csr, rp, ed, V, P, roots, depth, max_walks, "hub trees")
    assert counts.max() > 60


@pytest.mark.parametrize("depth,max_walks", [(0, 1), (1, 3), (2, 7), (3, 64), (4, 1000)])
def test_unused_rows_are_filled(depth, max_walks, monkeypatch):
    # outputs allocated by the binding: -1 and 0 past every root's walks, whatever the memory held
    say(f"[bfs] unused rows depth={depth} max_walks={max_walks}")
    rng = np.random.default_rng(depth)
    V, P, T = 700, 5, 1500
    s, p, o = rng.integers(0, V // 2, T), rng.integers(0, P, T), rng.integers(0, V, T)
    csr = gpu_csr(*(x.astype(np.int32) for x in (s, p, o)), V, P)
    roots = np.concatenate([rng.integers(0, V, 300), [V + 5, 0, -1]]).astype(np.int32)
    empty, filled = torch.empty, []

    def junk(*args, **kw):  # every buffer that the call allocates starts as junk
        filled.append(empty(*args, **kw).fill_(77))
        return filled[-1]

    d_roots, st = to_dev(roots), new_status()
    with monkeypatch.context() as m:
        m.setattr(torch, "empty", junk)
        tok, ln, cnt = rd.rdf2v_bfs_walks(csr, d_roots, depth, max_walks, status=st)
    assert any(x is tok for x in filled) and any(x is ln for x in filled)
    tok, ln, cnt = tok.cpu().numpy(), ln.cpu().numpy(), cnt.cpu().numpy()
    unused = np.arange(max_walks)[None, :] >= cnt[:, None]
    assert (tok[unused] == -1).all() and (ln[unused] == 0).all()
    assert (ln[~unused] > 0).all() and (tok[~unused][:, 0] >= 0).all()


@pytest.mark.parametrize("V,E,depth", [
    (1_200, 300_000, 2),       # an LDS tier: 600 rows, all of them the whole record array
    (1_200, 300_000, 4),
    (20, 300_000, 3),          # as few entities as one alignment unit of the workspace holds
    (1_200, 1_500_000, 3),     # rows longer than a tier expands: the bitmap pass
    (10_000, 1 << 20, 3),      # bitmap in LDS; 5,000 rows hold more than 2^32 records between them
    (1_400_000, 1 << 20, 3),   # bitmap in the workspace
])
def test_overlapping_rows_end_their_roots(V, E, depth):
    # row_ptr = 0, E, 0, E, ...: the rows of even entities are in range but all the same, those of
    # odd entities run backwards and no record leads to them. A level of many even entities has
    # more pairs than there are records, past 31 and 32 bits: its root ends with the status bit.
    say(f"[bfs] overlapping rows V={V} E={E} depth={depth}")
    rng = np.random.default_rng(V + E + depth)
    row_ptr = torch.tensor([0, E], dtype=torch.int32, device=device()).repeat(V // 2 + 1)[:V + 1].contiguous()
    edges = to_dev(np.stack([rng.integers(0, 3, E), 2 * rng.integers(0, V // 2, E)], axis=1))
    csr = rd.Csr(row_ptr, edges, V, 3)
    roots = 2 * np.arange(min(40, V // 2), dtype=np.int32)
    max_walks, guard = 16, 64
    width = 2 * depth + 1
    tok = torch.full((len(roots) * max_walks * width + 2 * guard,), -9, dtype=torch.int32, device=device())
    ln = torch.full((len(roots) * max_walks + 2 * guard,), -9, dtype=torch.int32, device=device())
    st = new_status()
    _, _, cnt = rd.rdf2v_bfs_walks(csr, to_dev(roots), depth, max_walks, tokens=tok[guard:-guard], lens=ln[guard:-guard],
                                   status=st)
    torch.cuda.synchronize()
    assert int(st.item()) & rd.RDF2V_STATUS_BAD_CSR
    assert bool((cnt >= 0).all()) and bool((cnt <= max_walks).all())
    for buf in (tok, ln):
        assert bool((buf[:guard] == -9).all()) and bool((buf[-guard:] == -9).all())


@pytest.mark.parametrize("V", [12, 900])
def test_rows_longer_than_a_tier_expands(V):
    # a consistent graph in which three entities have rows of 1.4M records, around the longest row
    # that an LDS tier takes: as root, below the root and at the depth limit
    say(f"[bfs] rows of 1.4M records, V={V}")
    P, far = 4, V - 3
    rng = np.random.default_rng(V)
    limit = (1 << 30) // 768
    sizes = {0: limit + 1, 7: limit, far: limit + 2}
    s = np.concatenate([np.full(n, v) for v, n in sizes.items()] + [rng.integers(1, V, 4 * V), [3, 3, 5]]).astype(np.int32)
    o = rng.integers(0, V - 2, len(s)).astype(np.int32)
    o[-3:] = (far, 4, 7)
    p = rng.integers(0, P, len(s)).astype(np.int32)
    rp, ed = oracle.build_csr(s, p, o, V, P)
    csr = gpu_csr(s, p, o, V, P)
    roots = np.array([3, 0, 5, far, 7, V - 1, 3], np.int32)
    for depth in (1, 2, 3):
        _compare(csr, rp, ed, V, P, roots, depth, V, f"long rows depth {depth}")
        _compare(csr, rp, ed, V, P, roots, depth, 5, f"long rows depth {depth} truncated")


@pytest.mark.parametrize("roots,max_walks,width,offset", [
    (1, 100_000, 9, 1), (3, 30_001, 5, 2), (70, 2_000, 7, 3),   # several workgroups to a root
    (1, 1, 1, 0), (300, 2, 3, 1), (1001, 7, 5, 2),              # several roots to a workgroup
    (40, 300, 3, 3), (500, 129, 17, 1), (9, 1, 129, 2),         # about a workgroup to a root
    (40, 50_001, 17, 3), (150_000, 75, 3, 1),                   # more than the Infinity Cache takes
])
def test_fill_unused_writes_the_unused_rows_only(roots, max_walks, width, offset):
    # outputs that begin anywhere in a 16-byte group, with ints around them that stay as they are
    say(f"[bfs] fill {roots} roots x {max_walks} rows of {width}")
    rng = np.random.default_rng(roots + max_walks + width)
    counts = rng.integers(0, max_walks + 1, roots).astype(np.int32)
    counts[rng.random(roots) < 0.2] = max_walks
    for k, odd in enumerate((-3, 0, max_walks + 5, max_walks)):  # outside [0, max_walks]: as clamped
        if k < roots:
            counts[k * 7 % roots] = odd
    guard = 8
    tok = torch.full((roots * max_walks * width + 2 * guard + offset,), -9, dtype=torch.int32, device=device())
    ln = torch.full((roots * max_walks + 2 * guard + offset,), -9, dtype=torch.int32, device=device())
    a, b = guard + offset, guard
    st = rd._native().rdf2v_bfs_fill_unused(to_dev(counts).data_ptr(), roots, max_walks, width, tok[a:].data_ptr(),
                                            ln[a:].data_ptr(), torch.cuda.current_stream().cuda_stream)
    assert st == rd.RDF2V_OK
    unused = np.arange(max_walks)[None, :] >= np.clip(counts, 0, max_walks)[:, None]
    ref_t = np.where(unused[:, :, None], -1, np.full((1, 1, width), -9)).reshape(-1)
    ref_l = np.where(unused, 0, -9).reshape(-1)
    for buf, ref in ((tok.cpu().numpy(), ref_t), (ln.cpu().numpy(), ref_l)):
        assert np.array_equal(buf[a:len(buf) - b], ref)
        assert (buf[:a] == -9).all() and (buf[len(buf) - b:] == -9).all()
