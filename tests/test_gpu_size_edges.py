"""Sizes at which the kernel of a call changes: the LDS chain's classes (1024,
2048, 4096 and 6144 edges, ids of 16 bits or more), the graphs after them, the
tile of a radix pass (2^17 records: at m for the permutation, at 2m for its
tuples), the finisher's list in LDS (16384 switches), and batches whose graphs
stop after different numbers of supersteps.  Exact against the oracle."""
import numpy as np
import pytest

import graphgen
import oracle

pytestmark = pytest.mark.gpu

torch = pytest.importorskip("torch")


def to_dev(E):
    return torch.from_numpy(np.ascontiguousarray(E, dtype=np.uint64).view(np.int64).copy()).to("cuda")


@pytest.fixture(scope="module", params=[60000, 70000], ids=["ids16", "ids32"])
def pool(request):
    return request.param, graphgen.gnp(request.param, 6.0 / request.param, 5)


@pytest.mark.parametrize("m", [1024, 1025, 2047, 2048, 2049, 4095, 4096, 4097, 6143, 6144, 6145, 8193, 32767, 32769,
                               65535, 65536, 65537, 131071, 131072, 131073])
@pytest.mark.parametrize("pl", [0, 1 << 29])
def test_size_edges_exact(pool, m, pl):
    if not torch.cuda.is_available():
        pytest.skip("no GPU")
    import paper_2111_03005_amd as gesmc
    n, P = pool
    E = np.random.default_rng(m).permutation(P)[:m]
    print("case edges n=%d m=%d pl=%d" % (n, m, pl), flush=True)
    c = gesmc.Context(0)
    try:
        out, st, steps = c.run(to_dev(E), n, 8, t0=2, r=3, pl=pl, steps=True)
        rc, exp, counts, _ = oracle.run(E, n, 8, 2, 3, pl)
        assert rc == 0
        assert np.array_equal(out.cpu().numpy().view(np.uint64), exp)
        for s, want in zip(steps, counts):
            assert all(s[k] == want[k] for k in ("attempts", "legal", "rej_loop", "rej_exists", "rej_pl"))
    finally:
        c.close()


# graphs above the LDS chain's sizes, so that they share a superstep's passes
@pytest.mark.parametrize("sizes", [(6500, 7000), (9001, 6147, 6999, 12000), (40001, 6500, 30000)])
@pytest.mark.parametrize("rs", [(1, 3, 2, 5), (4, 4, 4, 4), (3, 0, 1, 1)])
def test_batch_uneven_steps(pool, sizes, rs):
    if not torch.cuda.is_available():
        pytest.skip("no GPU")
    import paper_2111_03005_amd as gesmc
    n, P = pool
    gs = [np.random.default_rng(m).permutation(P)[:m] for m in sizes]
    rs = rs[:len(gs)]
    print("case batch n=%d sizes=%s rs=%s" % (n, sizes, rs), flush=True)
    c = gesmc.Context(0)
    try:
        offs = np.concatenate([[0], np.cumsum([len(E) for E in gs])])
        out, _, _ = c.run_batch(to_dev(np.concatenate(gs)), offs, [n] * len(gs), list(range(len(gs))), list(rs),
                                t0=[1] * len(gs))
        got = out.cpu().numpy().view(np.uint64)
        for i, E in enumerate(gs):
            rc, exp, _, _ = oracle.run(E, n, i, 1, rs[i], 0)
            assert rc == 0
            assert np.array_equal(got[offs[i]:offs[i + 1]], exp)
    finally:
        c.close()


# without per-superstep records, so that up to 4096 edges (6144 with 16-bit ids)
# run in the LDS chain; r = 35 takes two pieces of permutations
@pytest.mark.parametrize("m", [1, 2, 3, 511, 512, 513, 1023, 1024, 1025, 2047, 2048, 2049, 4095, 4096, 4097, 6143, 6144,
                               6145])
@pytest.mark.parametrize("pl,r", [(0, 3), (1 << 29, 35)])
def test_lds_chain_classes_exact(pool, m, pl, r):
    if not torch.cuda.is_available():
        pytest.skip("no GPU")
    import paper_2111_03005_amd as gesmc
    n, P = pool
    E = np.random.default_rng(m + 1).permutation(P)[:m]
    print("case LDS n=%d m=%d pl=%d r=%d" % (n, m, pl, r), flush=True)
    c = gesmc.Context(0)
    try:
        out, st = c.run(to_dev(E), n, 9, t0=4, r=r, pl=pl)
        rc, exp, counts, _ = oracle.run(E, n, 9, 4, r, pl)
        assert rc == 0
        assert np.array_equal(out.cpu().numpy().view(np.uint64), exp)
        assert all(st[k] == sum(x[k] for x in counts) for k in ("attempts", "legal", "rej_loop", "rej_exists", "rej_pl"))
        chain = 2 <= m <= (6144 if n <= 1 << 16 else 4096)
        assert (st["rounds_sum"] == 0) == (chain or m < 2)  # (the chain records no rounds)
    finally:
        c.close()


# few vertices: most targets present, so long lists, every class of the chain
@pytest.mark.parametrize("m", [900, 1024, 1900, 2048, 3900, 4096, 6000, 6144])
@pytest.mark.parametrize("wide", [False, True])
def test_lds_chain_dense_exact(m, wide):
    if not torch.cuda.is_available():
        pytest.skip("no GPU")
    import paper_2111_03005_amd as gesmc
    k = int((2.2 * m) ** 0.5) + 2
    E = np.random.default_rng(m).permutation(graphgen.gnp(k, 1.0, 1))[:m]
    n = k
    if wide:  # ids beyond 2^16
        E, n = (E + np.uint64((70000 << 32) | 70000)).astype(np.uint64), 70000 + k
    assert len(E) == m
    print("case dense LDS n=%d m=%d" % (n, m), flush=True)
    c = gesmc.Context(0)
    try:
        out, st = c.run(to_dev(E), n, 3, t0=1, r=12)
        rc, exp, counts, _ = oracle.run(E, n, 3, 1, 12, 0)
        assert rc == 0
        assert np.array_equal(out.cpu().numpy().view(np.uint64), exp)
        assert all(st[q] == sum(x[q] for x in counts) for q in ("attempts", "legal", "rej_loop", "rej_exists"))
    finally:
        c.close()
