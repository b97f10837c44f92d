"""Every buffer that a call takes from a caller's allocator is written within its
size: the allocator here hands out blocks with a guard behind each and looks at
the guards when a block comes back.  Odd sizes, so that each array ends off its
alignment."""
import numpy as np
import pytest

import graphgen
import oracle

pytestmark = pytest.mark.gpu

torch = pytest.importorskip("torch")

GUARD = 1 << 16


def to_dev(E):
    return torch.from_numpy(np.ascontiguousarray(E, dtype=np.uint64).view(np.int64).copy()).to("cuda")


class Guarded:
    def __init__(self):
        self.live, self.bad = {}, []

    def alloc(self, n):
        t = torch.full((n + GUARD + 256,), 0xA5, dtype=torch.uint8, device="cuda")
        p = (t.data_ptr() + 255) & ~255
        self.live[p] = (t, n, p - t.data_ptr())
        torch.cuda.synchronize()
        return p

    def check(self):
        torch.cuda.synchronize()
        for p, (t, n, off) in self.live.items():
            hit = torch.nonzero(t[off + n:off + n + GUARD] != 0xA5)
            if hit.numel():
                self.bad.append((n, int(hit.max()) + 1))

    def free(self, p):
        t, n, off = self.live.pop(p)
        hit = torch.nonzero(t[off + n:off + n + GUARD] != 0xA5)
        if hit.numel():
            self.bad.append((n, int(hit.max()) + 1))


def graphs():
    yield graphgen.gnp(33, 0.5, 1), 33
    yield graphgen.gnp(92, 0.1, 6)[-289:], 92
    yield graphgen.gnp(257, 0.3, 2)[:4097], 257
    yield graphgen.gnp(999, 0.04, 3), 999
    yield graphgen.powerlaw_graph(20011, 2.05, 1, 9000, 4), 20011
    yield graphgen.gnp(70001, 3e-5, 5), 70001


CALLS = {
    "run": lambda c, d, n: c.run(d, n, 3, t0=1, r=3),
    "steps": lambda c, d, n: c.run(d, n, 3, t0=1, r=3, steps=True),
    "class": lambda c, d, n: [c.run_class(d, n, 3, cls, 0, 3, outcomes=True) for cls in (1, 3, 4)],
    "batch": lambda c, d, n: c.run_batch(torch.cat([d, d[:7], d]), [0, d.numel(), d.numel() + 7, 2 * d.numel() + 7],
                                         [n] * 3, [1, 2, 3], [3, 1, 2]),
    "es": lambda c, d, n: [c.run_es(d, n, 3, r=r, outcomes=True) for r in (3, 3 * d.numel())],
    "mixing": lambda c, d, n: [c.mixing(d, n, 3, K, thin, chain=chain) for chain in (0, 1) for K, thin in
                               ((3, [1, 2]), (17, list(range(1, 17)))) if n <= 1000],
    "generators": lambda c, d, n: [c.gen_gnp(n, 2.5 / n, 5), c.gen_relabel(d.clone(), n, 3),
                                   c.gen_havel_hakimi(c.gen_pld_degrees(n, 2.3, 1, max(2, int(n ** 0.5)), 3)[0])],
    "hooks": lambda c, d, n: [c.permutation(d.numel(), 3, 1), c.perm_keys(d.numel(), 3, 1),
                              c.superstep_outcomes(d, n, 3, 1)],
}


@pytest.mark.parametrize("strategy", [0, 1])
@pytest.mark.parametrize("name", list(CALLS))
def test_buffers_written_within_their_sizes(name, strategy):
    if not torch.cuda.is_available():
        pytest.skip("no GPU")
    import paper_2111_03005_amd as gesmc
    for E, n in graphs():
        if strategy and name == "batch":
            continue  # (needs strategy 0)
        print("case guarded %s strategy %d: m=%d n=%d" % (name, strategy, len(E), n), flush=True)
        a = Guarded()
        c = gesmc.Context(0)
        c.set_option(gesmc.OPT_STRATEGY, strategy)
        c.set_allocator(a.alloc, a.free)
        CALLS[name](c, to_dev(E), n)
        a.check()
        assert not a.bad, "(size, bytes beyond it): %s" % a.bad
        rc, exp, _, _ = oracle.run(E, n, 5, 0, 2, 0)  # and the context goes on
        assert rc == 0 and np.array_equal(c.run(to_dev(E), n, 5, r=2)[0].cpu().numpy().view(np.uint64), exp)
        c.close()
        assert not a.bad and not a.live
