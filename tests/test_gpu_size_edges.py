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
