"""The caller-supplied allocator (gesmc_set_allocator): results identical to
the context's own hipMalloc buffers, every buffer returned to the allocator
that made it, and an allocation failure injected through the hook fails the
call cleanly (GESMC_E_NOMEM, output untouched, context usable afterwards)."""
import numpy as np
import pytest

import graphgen
import oracle

pytestmark = pytest.mark.gpu

torch = pytest.importorskip("torch")


def _gpu():
    if not torch.cuda.is_available():
        pytest.skip("no GPU")
    import paper_2111_03005_amd as gesmc
    return gesmc


def to_dev(E):
    return torch.from_numpy(np.ascontiguousarray(E, dtype=np.uint64).view(np.int64).copy()).to("cuda")


class Counting:
    """PyTorch's caching allocator with counts; fail_after = n makes the
    (n+1)-th allocation return no memory."""

    def __init__(self, fail_after=None):
        self.live, self.allocs, self.frees, self.fail_after = {}, 0, 0, fail_after

    def alloc(self, n):
        if self.fail_after is not None and self.allocs >= self.fail_after:
            return 0
        p = torch.cuda.caching_allocator_alloc(n, device=0)
        self.live[p] = n
        self.allocs += 1
        return p

    def free(self, p):
        assert p in self.live, "freed a buffer this allocator did not make"
        del self.live[p]
        self.frees += 1
        torch.cuda.caching_allocator_delete(p)


def test_torch_allocator_same_results_and_all_returned():
    gesmc = _gpu()
    E, n = graphgen.workload_powerlaw_1m()
    a = Counting()
    ctx = gesmc.Context(0)
    ctx.set_allocator(a.alloc, a.free)
    out, st = ctx.run(to_dev(E), n, 42, t0=0, r=2)
    ref = gesmc.Context(0)
    want, _ = ref.run(to_dev(E), n, 42, t0=0, r=2)
    assert torch.equal(out, want)
    assert a.allocs > 0 and len(a.live) == a.allocs - a.frees
    # batched and the generators allocate through it too
    g = graphgen.batch_graphs(8, 3, 1e2, 1e4)
    Eb, offs, ns = graphgen.concat(g)
    got_b, _, _ = ctx.run_batch(to_dev(Eb), offs, ns, [5 + q for q in range(8)], [3] * 8)
    want_b, _, _ = ref.run_batch(to_dev(Eb), offs, ns, [5 + q for q in range(8)], [3] * 8)
    assert torch.equal(got_b, want_b)
    G = ctx.gen_gnp(3000, 0.01, 7)
    assert np.array_equal(G.cpu().numpy().view(np.uint64), oracle.gen_gnp(3000, 0.01, 7))
    ctx.close()
    ref.close()
    assert a.live == {} and a.frees == a.allocs


def test_allocation_failure_through_the_hook():
    gesmc = _gpu()
    E, n = graphgen.gnp(20000, 0.001, 4), 20000
    a = Counting(fail_after=2)
    ctx = gesmc.Context(0)
    ctx.set_option(gesmc.OPT_SMALL_GRAPHS, 0)
    ctx.set_allocator(a.alloc, a.free)
    out = torch.full((len(E),), -1, dtype=torch.int64, device="cuda")
    with pytest.raises(gesmc.GesmcError) as ei:
        ctx.run(to_dev(E), n, 1, r=2, out=out)
    assert ei.value.status == gesmc.E_NOMEM
    assert (out == -1).all()
    a.fail_after = None  # the allocator recovers: the same context works
    got, _ = ctx.run(to_dev(E), n, 1, r=2, out=out)
    rc, want, _, _ = oracle.run(E, n, 1, 0, 2)
    assert np.array_equal(got.cpu().numpy().view(np.uint64), want)
    ctx.set_allocator(None, None)  # back to hipMalloc; earlier buffers keep their allocator
    got2, _ = ctx.run(to_dev(E), n, 1, r=2)
    assert torch.equal(got, got2)
    ctx.close()
    assert a.live == {}


def test_allocator_argument_checks():
    gesmc = _gpu()
    ctx = gesmc.Context(0)
    lib = gesmc._binding.load_library()
    from paper_2111_03005_amd._binding import ALLOC_FN, FREE_FN
    st = lib.gesmc_set_allocator(ctx._h, ALLOC_FN(lambda n, u: 0), FREE_FN(), None)
    assert st == gesmc.E_INVAL
    srv = gesmc.Server(ctx, hbm_budget_bytes=1 << 26)
    a = Counting()
    with pytest.raises(gesmc.GesmcError) as ei:
        ctx.set_allocator(a.alloc, a.free)  # not while a server uses the context
    assert ei.value.status == gesmc.E_INVAL
    srv.close()
    ctx.set_allocator(a.alloc, a.free)
    ctx.close()


class Refusing(Counting):
    """Returns no memory for the k-th allocation alone."""

    def __init__(self, k):
        super().__init__()
        self.k, self.asked = k, 0

    def alloc(self, n):
        self.asked += 1
        return 0 if self.asked - 1 == self.k else super().alloc(n)


def test_es_without_memory_for_windows():
    """Only the edge list, its slots, the edge set and the counters are needed:
    without memory for the windows (asked for last) the call runs on one workgroup."""
    gesmc = _gpu()
    n, m, r = 60000, 20000, 12000
    E = np.random.default_rng(1).permutation(graphgen.gnp(n, 6.0 / n, 5))[:m]
    rc, want, cnt, _ = oracle.es_run(E, n, 3, 0, r)
    assert rc == 0
    for k in range(5):
        print("case allocation %d refused" % k, flush=True)
        a = Refusing(k)
        ctx = gesmc.Context(0)
        ctx.set_allocator(a.alloc, a.free)
        out = torch.full((m,), -1, dtype=torch.int64, device="cuda")
        if k < 4:
            with pytest.raises(gesmc.GesmcError) as ei:
                ctx.run_es(to_dev(E), n, 3, r=r, out=out)
            assert ei.value.status == gesmc.E_NOMEM and (out == -1).all()
        for _ in range(1 if k == 4 else 2):  # (a failed call's context works, with windows or without)
            _, st = ctx.run_es(to_dev(E), n, 3, r=r, out=out)
            assert np.array_equal(out.cpu().numpy().view(np.uint64), want)
            assert all(st[q] == cnt[q] for q in ("attempts", "legal", "rej_loop", "rej_exists"))
        assert a.asked > 4
        ctx.close()
        assert a.live == {}


def test_mixing_block_goes_back():
    """The diagnostic's block (12 bytes a vertex pair and thinning value) is not
    kept from a caller's allocator, and gesmc_set_allocator returns a kept one."""
    gesmc = _gpu()
    n = 6000
    E = graphgen.gnp(n, 0.001, 3)
    counters = 12 * (n * (n - 1) // 2)
    a = Counting()
    ctx = gesmc.Context(0)
    d = to_dev(E)
    want, _ = ctx.mixing(d, n, 1, 4, [1, 2])  # kept by the context
    torch.cuda.synchronize()
    free0 = torch.cuda.mem_get_info()[0]
    ctx.set_allocator(a.alloc, a.free)
    assert torch.cuda.mem_get_info()[0] - free0 >= 2 * counters
    for _ in range(2):
        got, _ = ctx.mixing(d, n, 1, 4, [1, 2])
        assert got == want
        assert sum(a.live.values()) < counters
    ctx.close()
    assert a.live == {}


class RefusingSize(Counting):
    """Returns no memory for allocations of one size."""

    def __init__(self, size=None):
        super().__init__()
        self.size, self.sizes = size, []

    def alloc(self, n):
        self.sizes.append(n)
        return 0 if n == self.size else super().alloc(n)


@pytest.mark.parametrize("form", ["run", "class", "batch", "batch_graph"])
def test_each_buffer_refused(form):
    """Without memory for one of its buffers a call fails cleanly or, where the
    buffer only joins two passes into one, gives the same result with them apart."""
    gesmc = _gpu()
    n, r = 20000, 3
    E = graphgen.gnp(n, 0.001, 4)
    rc, want, _, _ = oracle.run(E, n, 1, 0, r)
    assert rc == 0
    stream = torch.cuda.Stream()

    def call(a):
        ctx = gesmc.Context(0)
        try:
            ctx.set_option(gesmc.OPT_GRAPH, 1 if form == "batch_graph" else 0)
            ctx.set_allocator(a.alloc, a.free)
            d, out = to_dev(E), torch.full((len(E),), -1, dtype=torch.int64, device="cuda")
            for _ in range(4 if form == "batch_graph" else 1):
                try:
                    if form == "run":
                        ctx.run(d, n, 1, r=r, out=out)
                    elif form == "class":
                        ctx.run_class(d, n, 1, 0, 0, r, out=out)
                    else:
                        with torch.cuda.stream(stream):
                            ctx.run_batch(d, [0, len(E)], [n], [1], [r], out=out, stream=stream)
                        stream.synchronize()
                except gesmc.GesmcError as e:
                    assert e.status == gesmc.E_NOMEM and (out == -1).all()
                    return False
                assert np.array_equal(out.cpu().numpy().view(np.uint64), want)
                out.fill_(-1)
                torch.cuda.synchronize()
            return True
        finally:
            ctx.close()
            assert a.live == {}

    a = RefusingSize()
    assert call(a)
    survived = 0
    for size in sorted(set(a.sizes)):
        print("case %s without %d bytes" % (form, size), flush=True)
        survived += call(RefusingSize(size))
    assert survived > 0
