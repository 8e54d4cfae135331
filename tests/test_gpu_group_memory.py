"""What a group call allocates for theta spread over all workgroups: nothing for
launches that cannot be spread, and no call is refused for it."""
import numpy as np
import pytest

import synth
from tests.gpu_util import have_gpu

pytestmark = [pytest.mark.gpu, pytest.mark.skipif(not have_gpu(), reason="no GPU")]


def _context(seed, n):
    import torch
    import paper_2501_12928_amd as eor
    inst = synth.small(seed=seed, m=n + 40, n=n, n_k=1, n_theta=1)
    return eor.Context(0).precompute(torch.from_numpy(inst.T).cuda(), torch.from_numpy(inst.noise_var).cuda(),
                                     torch.from_numpy(inst.d).cuda(), 1, inst.bin_of, inst.fixed_var)


def test_no_call_refused_for_the_spread_route():
    """Five million small theta beside one at n = 4096. The estimates prefer the
    spread route, whose arrays for all of them (64 KiB of solve vectors each at
    the largest instance's size: 328 GB) no device holds; the route with one
    workgroup per theta needs a slot per resident workgroup."""
    import torch
    import paper_2501_12928_amd as eor
    B = 5_000_000
    ctxs = [_context(1, 4096), _context(2, 40)]
    g = torch.Generator(device="cuda").manual_seed(3)
    th = [-1.0 + 4.0 * torch.rand(b, 1, dtype=torch.float64, device="cuda", generator=g) for b in (1, B)]
    grp = eor.Group(ctxs)
    print(f"gpu: group of 1 + {B} theta", flush=True)
    outs, infos = grp.loglike(th)
    torch.cuda.synchronize()
    assert all(bool((i == 0).all()) for i in infos)
    for c, t, o in zip(ctxs, th, outs):
        print(f"gpu: {t.shape[0]} theta of one context", flush=True)
        assert torch.equal(c.loglike_batch(t)[0], o)
    grp.close()
    for c in ctxs:
        c.close()


def test_spread_memory_follows_each_theta_s_size():
    """Batch sizes that change from call to call, small theta beside a large one:
    every theta's bits are those of its own context, and the solve vectors of
    4000 more small theta take what those theta need (4 KiB of solve vector and
    progress words each at most), not the largest instance's size."""
    import torch
    import paper_2501_12928_amd as eor
    ctxs = [_context(11, 2048), _context(12, 40), _context(13, 100)]
    gen = torch.Generator(device="cuda").manual_seed(14)
    th = [-1.0 + 4.0 * torch.rand(b, 1, dtype=torch.float64, device="cuda", generator=gen) for b in (2, 4500, 60)]
    alone = [c.loglike_batch(t)[0] for c, t in zip(ctxs, th)]
    outs = [torch.empty_like(a) for a in alone]
    infos = [torch.empty(a.shape, dtype=torch.int32, device="cuda") for a in alone]
    grp = eor.Group(ctxs)
    used = None
    for sizes in ((1, 500, 7), (1, 4500, 7), (2, 300, 60), (0, 20, 3), (2, 4500, 60), (1, 500, 7)):
        print(f"gpu: group of {sizes} theta", flush=True)
        for o in outs:
            o.fill_(7.0)
        grp.loglike([t[:b] for t, b in zip(th, sizes)], outs=outs, infos=infos)
        torch.cuda.synchronize()
        for a, o, b in zip(alone, outs, sizes):
            assert torch.equal(o[:b], a[:b]) and bool((o[b:] == 7.0).all())
        free = torch.cuda.mem_get_info()[0]
        if used is None:
            used = free
        else:
            # the allocator hands out 2 MiB pieces: one more for each of four buffers
            assert used - free <= 4000 * 4096 + (8 << 20), (used - free, sizes)
    grp.close()
    for c in ctxs:
        c.close()


def test_creating_a_group_does_not_wait_for_the_device():
    """A group is created while another stream has a second of work queued."""
    import torch
    import paper_2501_12928_amd as eor
    ctxs = [_context(21, 70), _context(22, 40)]
    gen = torch.Generator(device="cuda").manual_seed(23)
    th = [-1.0 + 4.0 * torch.rand(b, 1, dtype=torch.float64, device="cuda", generator=gen) for b in (3, 5)]
    alone = [c.loglike_batch(t)[0] for c, t in zip(ctxs, th)]
    torch.cuda.synchronize()
    side, done = torch.cuda.Stream(), torch.cuda.Event()
    print("gpu: a group beside a busy stream", flush=True)
    with torch.cuda.stream(side):
        torch.cuda._sleep(1_000_000_000)
        done.record()
    grp = eor.Group(ctxs)
    assert not done.query()
    torch.cuda.synchronize()
    outs, infos = grp.loglike(th)
    torch.cuda.synchronize()
    assert all(torch.equal(o, a) for o, a in zip(outs, alone))
    grp.close()
    for c in ctxs:
        c.close()
