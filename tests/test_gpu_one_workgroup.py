"""The kernel that gives each theta a workgroup of its own, with 64-wide tiles.
Calls of few theta are spread over all workgroups instead, so these take 512 theta
(5120 where there is one tile row), which never are (test_route.py holds the rule
to that)."""
import numpy as np
import pytest

import synth
from tests.gpu_util import have_gpu, tol

pytestmark = [pytest.mark.gpu, pytest.mark.skipif(not have_gpu(), reason="no GPU")]

# Launch choices (prefetch stages, workgroups per CU, tiles per pass).
TUNINGS = [(4, 1, 2), (2, 1, 2), (4, 2, 1), (2, 2, 1), (4, 1, 1)]


def _ctx(inst):
    import torch
    import paper_2501_12928_amd as eor
    return eor.Context(0).precompute(torch.from_numpy(inst.T).cuda(), torch.from_numpy(inst.noise_var).cuda(),
                                     torch.from_numpy(inst.d).cuda(), inst.n_k, inst.bin_of, inst.fixed_var)


def _many(n):
    return 512 if n > 64 else 5120


def _check(got, ref):
    assert np.all(np.abs(got - ref) <= np.minimum(tol(ref), 1e-10 * np.abs(ref)))


# 2 tile rows, whole and ragged; 3; 5, ragged by one; 11
@pytest.mark.parametrize("m,n,n_k", [(200, 128, 2), (300, 130, 4), (520, 257, 5), (900, 700, 6)])
def test_launch_choices_agree(orc, m, n, n_k):
    """Every launch choice gives the same bits, which are those of a call of a few
    theta, and meets the oracle."""
    import torch
    inst = synth.small(seed=m + n, m=m, n=n, n_k=n_k, n_theta=512)
    ref, _ = orc.loglike_instance(inst, theta=inst.theta[:4])
    t = torch.from_numpy(inst.theta).cuda()
    ctx = _ctx(inst)
    few = [x.clone() for x in ctx.loglike_terms(t[:9])]
    base = None
    for tuning in TUNINGS:
        print(f"gpu: 512 theta, n={n}, tuning {tuning}", flush=True)
        ctx.set_tuning(*tuning)
        L, info, terms = ctx.loglike_terms(t)
        assert not info.any()
        if base is None:
            base = (L.clone(), terms.clone())
            _check(L[:4].cpu().numpy(), ref)
            assert torch.equal(L[:9], few[0]) and torch.equal(terms[:9], few[2])
        assert torch.equal(L, base[0]) and torch.equal(terms, base[1]), tuning
    ctx.close()


@pytest.mark.parametrize("tuning", TUNINGS)
@pytest.mark.parametrize("n", [40, 100, 200])
def test_failures_reported_per_theta(orc, n, tuning):
    """Invalid theta among many valid ones: info -1 and logL -inf for those, and the
    others are the bits of a batch without them."""
    import torch
    B = _many(n)
    inst = synth.small(seed=n, m=n + 50, n=n, n_k=3, n_theta=B)
    th = inst.theta.copy()
    bad = {0: (2, np.nan), 7: (0, np.inf), 255: (1, -np.inf), 256: (1, 400.0), 300: (0, np.nan), B - 1: (2, -400.0)}
    for b, (k, v) in bad.items():
        th[b, k] = v
    ctx = _ctx(inst)
    ctx.set_tuning(*tuning)
    print(f"gpu: invalid theta among {B}, n={n}, tuning {tuning}", flush=True)
    good = ctx.loglike_batch(torch.from_numpy(inst.theta).cuda())[0].cpu().numpy()
    got, info = (x.cpu().numpy() for x in ctx.loglike_batch(torch.from_numpy(th).cuda()))
    rows = sorted(bad)
    _, rinfo = orc.loglike_instance(inst, theta=th[rows])
    np.testing.assert_array_equal(info[rows], rinfo)
    assert np.all(info[rows] == -1) and np.all(got[rows] == -np.inf)
    ok = np.ones(B, dtype=bool)
    ok[rows] = False
    assert not info[ok].any()
    np.testing.assert_array_equal(got[ok], good[ok])
    ctx.close()


@pytest.mark.parametrize("tuning", TUNINGS)
def test_failed_pivots(tuning):
    """A NaN column of T fails every theta at its own pivot, wherever it lies in the
    16-wide blocks and 64-wide tiles, and the next call on the context is as before."""
    import torch
    good = synth.small(seed=71, m=260, n=200, n_k=3, n_theta=512)
    t = torch.from_numpy(good.theta).cuda()
    ctx = _ctx(good)
    ctx.set_tuning(*tuning)
    ref = ctx.loglike_batch(t)[0].clone()
    rest = [torch.from_numpy(x).cuda() for x in (good.noise_var, good.d)]
    for col in (0, 1, 15, 16, 47, 48, 63, 64, 79, 127, 128, 191, 192, 199):
        T = torch.from_numpy(good.T).cuda()
        T[:, col] = float("nan")
        print(f"gpu: NaN column {col}, tuning {tuning}", flush=True)
        ctx.precompute(T, *rest, good.n_k, good.bin_of, good.fixed_var)
        L, info = ctx.loglike_batch(t)
        assert bool((info == col + 1).all()) and bool((L == -float("inf")).all())
    ctx.precompute(torch.from_numpy(good.T).cuda(), *rest, good.n_k, good.bin_of, good.fixed_var)
    assert torch.equal(ctx.loglike_batch(t)[0], ref)
    ctx.close()


@pytest.mark.parametrize("n", [1, 15, 16, 17, 33, 48, 49, 63, 64, 65, 80, 81, 97, 112, 113, 127, 129])
def test_padded_blocks_are_left_out(orc, n):
    """The 16-wide blocks of the last tile that hold only padding are not eliminated."""
    import torch
    inst = synth.small(seed=93, m=2 * n + 20, n=n, n_k=1, n_theta=_many(n))
    ref, _ = orc.loglike_instance(inst, theta=inst.theta[:3])
    ctx = _ctx(inst)
    print(f"gpu: n={n}, {_many(n)} theta", flush=True)
    L, info = ctx.loglike_batch(torch.from_numpy(inst.theta).cuda())
    assert not info.any()
    _check(L[:3].cpu().numpy(), ref)
    ctx.close()


@pytest.mark.parametrize("n", [5, 40, 64])
def test_one_tile_row_in_any_batch(n):
    """One tile row: calls that are spread, in one round or several, and calls that
    are not give the same bits."""
    import torch
    inst = synth.small(seed=n, m=n + 30, n=n, n_k=2, n_theta=5120)
    t = torch.from_numpy(inst.theta).cuda()
    ctx = _ctx(inst)
    print(f"gpu: n={n}, 5120 theta", flush=True)
    whole, info = ctx.loglike_batch(t)
    assert not info.any()
    for B in (1, 255, 256, 257, 1000, 3000):
        print(f"gpu: n={n}, {B} theta", flush=True)
        assert torch.equal(ctx.loglike_batch(t[:B])[0], whole[:B])
    ctx.close()


def test_group_with_many_theta():
    """A group with too many theta to be spread: four-wave and eight-wave workgroups,
    eager and from a graph, give each context's own bits; an invalid theta and a
    context whose pivot fails leave the others as they are."""
    import torch
    import paper_2501_12928_amd as eor
    shapes = [(70, 300), (150, 400), (257, 300), (300, 500), (64, 300), (500, 100), (33, 400), (130, 60)]
    insts = [synth.small(seed=400 + k, m=2 * n, n=n, n_k=2, n_theta=B) for k, (n, B) in enumerate(shapes)]
    insts[-1].T = insts[-1].T.copy()
    insts[-1].T[:, 99] = np.nan
    ctxs = [_ctx(i) for i in insts]
    th = [torch.from_numpy(i.theta).cuda() for i in insts]
    th[2][17, 0] = float("nan")
    own = [[x.clone() for x in c.loglike_batch(t)] for c, t in zip(ctxs, th)]
    assert own[2][1][17] == -1 and bool((own[-1][1] == 100).all())
    g = eor.Group(ctxs)
    outs = infos = None
    for graph in (False, True):
        g.set_graph(graph)
        for tuning in TUNINGS:
            print(f"gpu: group of {sum(b for _, b in shapes)} theta, graph {graph}, tuning {tuning}", flush=True)
            g.set_tuning(*tuning)
            for _ in range(2):
                outs, infos = g.loglike(th, outs=outs, infos=infos)
                torch.cuda.synchronize()
                for (L, info), o, f in zip(own, outs, infos):
                    assert torch.equal(f, info) and torch.equal(o, L)
                    o.fill_(3.0)
    g.close()
    for c in ctxs:
        c.close()
