"""Decision rounds on graphs whose switches nearly all depend on each other:
every workgroup then stages as many undecided switches as it can hold, every
key has many inserters of which one at most may win, and the finishing
workgroup takes many passes.  Exact against the oracle for every schedule."""
import numpy as np
import pytest

import graphgen
import oracle

pytestmark = pytest.mark.gpu

torch = pytest.importorskip("torch")


def to_dev(E):
    return torch.from_numpy(np.ascontiguousarray(E, dtype=np.uint64).view(np.int64).copy()).to("cuda")


# n, p: dense enough that most targets are present or proposed several times
@pytest.mark.parametrize("n,p", [(150, 0.6), (230, 0.5), (700, 0.9)])
@pytest.mark.parametrize("fast", [None, 0, 1, 6])
@pytest.mark.parametrize("pack,pl", [(1, 0), (0, 1 << 30)])
def test_dense_rounds_exact(n, p, fast, pack, pl):
    if not torch.cuda.is_available():
        pytest.skip("no GPU")
    import paper_2111_03005_amd as gesmc
    E = graphgen.gnp(n, p, 31 + n)
    print("case dense n=%d m=%d fast=%s pack=%d pl=%d" % (n, len(E), fast, pack, pl), flush=True)
    c = gesmc.Context(0)
    try:
        c.set_option(gesmc.OPT_PACK_TUPLES, pack)
        if fast is not None:
            c.set_option(gesmc.OPT_FAST_ROUNDS, fast)
        for t0 in (0, 4):  # the second call may adapt its rounds to the first
            out, st, steps = c.run(to_dev(E), n, 9, t0=t0, r=4, pl=pl, steps=True)
            rc, exp, counts, _ = oracle.run(E, n, 9, t0, 4, pl)
            assert rc == 0
            assert np.array_equal(out.cpu().numpy().view(np.uint64), exp)
            for s, want in zip(steps, counts):
                assert all(s[k] == want[k] for k in ("attempts", "legal", "rej_loop", "rej_exists", "rej_pl"))
    finally:
        c.close()
