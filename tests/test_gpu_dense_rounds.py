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


def alg1_rounds(E, n, seed, t):
    """The round of Alg. 1 in which each switch of superstep t is decided, if
    every round sees only what the rounds before it decided."""
    ell = len(E) // 2
    pi = np.asarray(oracle.permutation(len(E), seed, t)).astype(np.int64).tolist()
    rc, _, _, codes = oracle.run(E, n, seed, t, 1, 0, outcomes=True)
    assert rc == 0
    codes = np.asarray(codes).reshape(-1).tolist()
    uv = [(int(e) >> 32, int(e) & 0xFFFFFFFF) for e in E]
    eraser = {uv[i]: p // 2 if p < 2 * ell else ell for p, i in enumerate(pi)}
    inserters, rounds = {}, [0] * ell
    for k in range(ell):
        i, j = pi[2 * k], pi[2 * k + 1]
        (u, v), (x, y) = uv[i], uv[j]
        targets = ((u, y), (v, x)) if i < j else ((u, x), (v, y))
        if codes[k] == 2:
            continue
        present, known = [], [0]  # rounds that show a target present; rounds of all it depends on
        for a, b in targets:
            key = (min(a, b), max(a, b))
            e = eraser.get(key)
            if e is not None and (e >= k or codes[e] == 2):
                present.append(0)
            elif e is not None:
                known.append(rounds[e])
                if codes[e] != 1:
                    present.append(rounds[e])
            for q in inserters.get(key, ()):
                if e is None or q > e:
                    known.append(rounds[q])
                    if codes[q] == 1:
                        present.append(rounds[q])
            inserters.setdefault(key, []).append(k)
        assert (codes[k] == 1) == (not present)
        rounds[k] = 1 + (max(known) if codes[k] == 1 else min(present))
    return rounds


# undecided after round 1: about 1500 (the finisher's list in LDS) and 4200
# (from memory), three and nine passes of its workgroup
@pytest.mark.parametrize("n", [600, 1000])
def test_round_limit_counts_sweeps(n):
    """A limit of as many rounds as Alg. 1 needs is met, whatever number of
    passes the finishing workgroup takes for a round."""
    if not torch.cuda.is_available():
        pytest.skip("no GPU")
    import paper_2111_03005_amd as gesmc
    E = graphgen.gnp(n, 0.1, 31)
    need = max(alg1_rounds(E, n, 5, 0))
    assert 2 <= need <= 8  # (later sweeps are cut into chunks of switches)
    c = gesmc.Context(0)
    try:
        c.set_option(gesmc.OPT_FAST_ROUNDS, 0)
        rc, exp, _, _ = oracle.run(E, n, 5, 0, 1, 0)
        out, _, steps = c.run(to_dev(E), n, 5, r=1, steps=True)
        print("needs %d rounds, %d undecided, %d passes" % (need, steps[0]["undecided_after_round1"],
                                                            steps[0]["rounds"]), flush=True)
        assert steps[0]["rounds"] > need
        c.set_option(gesmc.OPT_ROUND_LIMIT, need)
        out, _, _ = c.run(to_dev(E), n, 5, r=1, steps=True)
        assert np.array_equal(out.cpu().numpy().view(np.uint64), exp)
        c.set_option(gesmc.OPT_ROUND_LIMIT, 1)
        sentinel = torch.full((len(E),), 7, dtype=torch.int64, device="cuda")
        with pytest.raises(gesmc.GesmcError) as ei:
            c.run(to_dev(E), n, 5, r=1, steps=True, out=sentinel)
        assert ei.value.status == gesmc.E_ROUNDS and bool((sentinel == 7).all())
    finally:
        c.close()


# the finisher's first sweep is shared by workgroups from 8193 switches on, if
# its list is longer than 1024, or 2048 up to 65536 switches; every form of call,
# with a hub-free call in between that leaves nothing to share
@pytest.mark.parametrize("m", [16385, 16386, 16388, 32767, 32768, 32770, 90001, 131070, 131073, 131074])
@pytest.mark.parametrize("p", [0.01, 0.04, 0.12, 0.5, 0.95])
def test_shared_sweep_exact(m, p):
    if not torch.cuda.is_available():
        pytest.skip("no GPU")
    import paper_2111_03005_amd as gesmc
    n = int((2.1 * m / p) ** 0.5) + 3
    E = np.random.default_rng(m).permutation(graphgen.gnp(n, p, 17))[:m]
    assert len(E) == m
    sparse = graphgen.gnp(30000, 1e-4, 2)
    c = gesmc.Context(0)
    try:
        c.set_option(gesmc.OPT_FAST_ROUNDS, 0)
        rc, exp, counts, codes = oracle.run(E, n, 6, 0, 3, 0, outcomes=True)
        rc2, exp_s, _, _ = oracle.run(sparse, 30000, 6, 0, 3, 0)
        assert rc == 0 and rc2 == 0
        for form in ("run", "sparse", "class", "batch", "mixed batch"):
            print("case shared m=%d p=%g %s" % (m, p, form), flush=True)
            if form == "run":
                out, st, steps = c.run(to_dev(E), n, 6, r=3, steps=True)
                print("undecided", [s["undecided_after_round1"] for s in steps], "passes", [s["rounds"] for s in steps],
                      flush=True)
                for s, want in zip(steps, counts):
                    assert all(s[k] == want[k] for k in ("attempts", "legal", "rej_loop", "rej_exists", "rej_pl"))
            elif form == "sparse":
                out, _ = c.run(to_dev(sparse), 30000, 6, r=3)
                assert np.array_equal(out.cpu().numpy().view(np.uint64), exp_s)
                continue
            elif form == "class":
                out, _, _, got = c.run_class(to_dev(E), n, 6, 0, 0, 3, outcomes=True)
                assert np.array_equal(got.cpu().numpy(), np.asarray(codes).reshape(-1))
            elif form == "batch":
                out, _, _ = c.run_batch(to_dev(E), [0, m], [n], [6], [3])
            else:
                both = np.concatenate([E, sparse])
                out, _, _ = c.run_batch(to_dev(both), [0, m, len(both)], [n, 30000], [6, 6], [3, 3])
                out = out.cpu()
                assert np.array_equal(out[m:].numpy().view(np.uint64), exp_s)
                out = out[:m]
            assert np.array_equal(out.cpu().numpy().view(np.uint64), exp)
    finally:
        c.close()
