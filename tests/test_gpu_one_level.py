"""Radix passes of one level, and run bases summed inside the scatter: sizes at
which a plan gains a bucket bit (bucket means halve at 1152 * 2^B records),
where the summed tiles reach their limit, odd edge counts and remainders of a
tile, against the oracle."""
import numpy as np
import pytest

import graphgen
import oracle

pytestmark = pytest.mark.gpu

torch = pytest.importorskip("torch")


def to_dev(E):
    return torch.from_numpy(np.ascontiguousarray(E, dtype=np.uint64).view(np.int64).copy()).to("cuda")


@pytest.fixture(scope="module")
def pool():
    return graphgen.gnp(60000, 28.0 / 59999, 12)


# m: one bucket; its limit and the next record; one and several tiles; the
# limits of one level (1152 << 10 tuple slots at m = 589824, records beyond)
@pytest.mark.parametrize("m", [1023, 1152, 1153, 2048, 2049, 4607, 9217, 36865, 147457, 294911, 294913, 589823,
                               589825, 700001])
@pytest.mark.parametrize("pack,fuse", [(1, 1), (0, 1), (0, 0)])
def test_one_level_exact(pool, m, pack, fuse):
    if not torch.cuda.is_available():
        pytest.skip("no GPU")
    import paper_2111_03005_amd as gesmc
    E = np.random.default_rng(m).permutation(pool)[:m]
    print("case one level m=%d pack=%d fuse=%d" % (m, pack, fuse), flush=True)
    c = gesmc.Context(0)
    try:
        c.set_option(gesmc.OPT_SMALL_GRAPHS, 0)
        c.set_option(gesmc.OPT_PACK_TUPLES, pack)
        c.set_option(gesmc.OPT_FUSE_EMIT, fuse)
        out, st, steps = c.run(to_dev(E), 60000, 3, t0=1, r=3, steps=True)
        rc, exp, counts, _ = oracle.run(E, 60000, 3, 1, 3, 0)
        assert rc == 0
        assert np.array_equal(out.cpu().numpy().view(np.uint64), exp)
        assert [s["legal"] for s in steps] == [x["legal"] for x in counts]
    finally:
        c.close()


# up to one bucket a permutation takes no radix pass; above it takes one
@pytest.mark.parametrize("m", [2, 300, 577, 1151, 1152, 1153, 1154, 2305])
def test_permutation_of_one_bucket(pool, m):
    if not torch.cuda.is_available():
        pytest.skip("no GPU")
    import paper_2111_03005_amd as gesmc
    E = np.random.default_rng(m).permutation(pool)[:m]
    print("case one bucket m=%d" % m, flush=True)
    c = gesmc.Context(0)
    try:
        c.set_option(gesmc.OPT_PROFILE, 1)
        got = c.permutation(m, 7, 3)
        assert np.array_equal(got.cpu().numpy().astype(np.uint64), oracle.permutation(m, 7, 3).astype(np.uint64))
        assert ("k_scatter1" in c.profile()) == (m > 1152)
        for cls in (0, 1, 3, 4):
            c.set_option(gesmc.OPT_SMALL_GRAPHS, 0)
            out, _, _, codes = c.run_class(to_dev(E), 60000, 3, cls, 1, 4, outcomes=True)
            rc, exp, _, oc = oracle.run_class(E, 60000, 3, 1, 4, 0, cls, outcomes=True)
            assert rc == 0 and np.array_equal(out.cpu().numpy().view(np.uint64), exp)
            assert np.array_equal(codes.cpu().numpy(), np.asarray(oc).reshape(-1))
    finally:
        c.close()
