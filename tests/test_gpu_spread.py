"""Theta spread over all workgroups against one workgroup per theta: the same
bits, whatever the batch a theta is in; failures; uneven groups. A call of 256
theta or more runs whole rounds of one workgroup per theta, a call of few theta
(more than one tile row) is spread."""
import numpy as np
import pytest

import synth
from tests.gpu_util import have_gpu, tol

pytestmark = [pytest.mark.gpu, pytest.mark.skipif(not have_gpu(), reason="no GPU")]


def _ctx(inst):
    import torch
    import paper_2501_12928_amd as eor
    ctx = eor.Context(0)
    return ctx.precompute(torch.from_numpy(inst.T).cuda(), torch.from_numpy(inst.noise_var).cuda(),
                          torch.from_numpy(inst.d).cuda(), inst.n_k, inst.bin_of, inst.fixed_var)


# one past a tile, whole tiles, ragged; 2, 3, 3, 5, 9 and 17 tile rows
@pytest.mark.parametrize("m,n", [(150, 65), (300, 129), (300, 192), (500, 300), (700, 520), (1300, 1030)])
def test_same_bits_in_any_batch(orc, m, n):
    import torch
    inst = synth.small(seed=n, m=m, n=n, n_k=4, n_theta=256)
    th = inst.theta.copy()
    th[5, 1] = np.nan
    th[17, 0] = np.inf
    ctx = _ctx(inst)
    t = torch.from_numpy(th).cuda()
    print(f"gpu: n={n}, 256 theta", flush=True)
    whole, info, terms = (x.cpu().numpy() for x in ctx.loglike_terms(t))
    assert np.flatnonzero(info).tolist() == [5, 17] and np.all(info[[5, 17]] == -1)
    ref, _ = orc.loglike_instance(inst, theta=th[:3])
    assert np.all(np.abs(whole[:3] - ref) <= np.minimum(tol(ref), 1e-10 * np.abs(ref)))
    at = 0
    for B in (1, 2, 7, 1, 16, 33, 1):   # the second call holds theta 1 and 2, the third theta 5, the fifth theta 17
        print(f"gpu: n={n}, {B} theta from {at}", flush=True)
        part, pinfo, pterms = (x.cpu().numpy() for x in ctx.loglike_terms(t[at:at + B]))
        np.testing.assert_array_equal(part, whole[at:at + B])
        np.testing.assert_array_equal(pinfo, info[at:at + B])
        np.testing.assert_array_equal(pterms, terms[at:at + B])
        at += B
    # a full round and a remainder in one call
    both = torch.cat([t, t[:20]])
    got, _ = ctx.loglike_batch(both)
    np.testing.assert_array_equal(got.cpu().numpy(), np.concatenate([whole, whole[:20]]))
    ctx.close()


@pytest.mark.parametrize("m,n,calls", [(500, 300, 400), (1300, 1030, 800)])
def test_same_bits_in_every_call(m, n, calls):
    """Tiles pass between workgroups on different XCDs: no call may see one
    before it is complete. (Where the write-back of a workgroup's L2 was not
    waited for, one theta in 4000 at n = 1030 differed.)"""
    import torch
    inst = synth.small(seed=n, m=m, n=n, n_k=4, n_theta=256)
    ctx = _ctx(inst)
    t = torch.from_numpy(inst.theta).cuda()
    print(f"gpu: n={n}, {calls} calls", flush=True)
    whole, _, terms = ctx.loglike_terms(t)
    rng = np.random.default_rng(n)
    for _ in range(calls):
        B = int(rng.integers(1, 24))
        at = int(rng.integers(0, 256 - B))
        part, info, pterms = ctx.loglike_terms(t[at:at + B])
        assert torch.equal(part, whole[at:at + B]) and torch.equal(pterms, terms[at:at + B])
        assert not info.any()
    ctx.close()


@pytest.mark.parametrize("col", [0, 63, 64, 130, 191, 192, 299])
def test_failed_pivot_then_good_call(col):
    """A pivot that fails in any tile column is reported for every theta, and
    the next call on the context starts clean."""
    import torch
    good = synth.small(seed=71, m=420, n=300, n_k=3, n_theta=5)
    bad = synth.small(seed=71, m=420, n=300, n_k=3, n_theta=5)
    bad.T = bad.T.copy()
    bad.T[:, col] = np.nan
    ctx = _ctx(good)
    t = torch.from_numpy(good.theta).cuda()
    ref = ctx.loglike_batch(t)[0].cpu().numpy()
    for _ in range(2):
        ctx.precompute(torch.from_numpy(bad.T).cuda(), torch.from_numpy(bad.noise_var).cuda(),
                       torch.from_numpy(bad.d).cuda(), bad.n_k, bad.bin_of, bad.fixed_var)
        print(f"gpu: NaN column {col}", flush=True)
        L, info = ctx.loglike_batch(t)
        assert np.all(info.cpu().numpy() == col + 1) and np.all(L.cpu().numpy() == -np.inf)
        ctx.precompute(torch.from_numpy(good.T).cuda(), torch.from_numpy(good.noise_var).cuda(),
                       torch.from_numpy(good.d).cuda(), good.n_k, good.bin_of, good.fixed_var)
        np.testing.assert_array_equal(ctx.loglike_batch(t)[0].cpu().numpy(), ref)
    ctx.close()


def test_uneven_group():
    """Few theta of uneven instances in one spread launch, one instance without
    theta: each theta's bits are those of its own context; then other batch
    sizes, with more theta than workgroups."""
    import torch
    import paper_2501_12928_amd as eor
    shapes = [(400, 3), (65, 4), (1000, 2), (640, 0), (700, 5), (30, 1)]
    insts = [synth.small(seed=500 + k, m=2 * n, n=n, n_k=3, n_theta=max(B, 1)) for k, (n, B) in enumerate(shapes)]
    ctxs = [_ctx(i) for i in insts]
    g = eor.Group(ctxs)
    for reps in (1, 2, 60):
        th = [torch.from_numpy(np.tile(i.theta, (reps, 1))[:B * reps]).cuda() for i, (_, B) in zip(insts, shapes)]
        print(f"gpu: uneven group, {reps} x the theta", flush=True)
        outs, infos = g.loglike(th)
        outs, infos = g.loglike(th, outs=outs, infos=infos)
        torch.cuda.synchronize()
        for c, t, o, f in zip(ctxs, th, outs, infos):
            if t.shape[0]:
                assert torch.equal(c.loglike_batch(t)[0], o) and bool((f == 0).all())
    g.close()
    for c in ctxs:
        c.close()
