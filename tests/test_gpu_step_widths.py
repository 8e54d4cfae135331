"""Loss and gradient at the widths where the training kernel changes between
eight and sixteen waves, and with only one of the two outputs asked for."""
import numpy as np
import pytest

from oracle import mlp
from tests.gpu_util import have_gpu

pytestmark = [pytest.mark.gpu, pytest.mark.skipif(not have_gpu(), reason="no GPU")]


@pytest.mark.parametrize("H,nb", [(252, 15), (256, 16), (260, 17), (384, 33), (388, 1), (508, 40)])
def test_widths_and_single_outputs(H, nb):
    import torch
    import paper_2501_12928_amd as eor
    n_in, M = 5, 2
    rng = np.random.default_rng(H)
    s = eor.Surrogate(n_in, -1.0, 3.0, n_members=M, hidden=H, seed=0)
    p32 = np.stack([mlp.he_init(rng, n_in, H) for _ in range(M)]).astype(np.float32)
    x = rng.uniform(-1, 1, size=(M, nb, n_in)).astype(np.float32)
    y = rng.standard_normal((M, nb)).astype(np.float32)
    s.set_params(p32)
    print(f"gpu: loss/grad H={H} nb={nb}", flush=True)
    loss, grad = s.loss_grad(x, y)
    xd, yd = torch.from_numpy(x).cuda(), torch.from_numpy(y).cuda()
    only_l, only_g = torch.full_like(loss, 7.0), torch.full_like(grad, 7.0)
    lib = eor.lib()
    assert lib.eor_surrogate_loss_grad(s._h, nb, xd.data_ptr(), yd.data_ptr(), only_l.data_ptr(), None, None) == 0
    assert lib.eor_surrogate_loss_grad(s._h, nb, xd.data_ptr(), yd.data_ptr(), None, only_g.data_ptr(), None) == 0
    torch.cuda.synchronize()
    assert torch.equal(only_l, loss) and torch.equal(only_g, grad)
    loss, grad = loss.cpu().numpy(), grad.cpu().numpy()
    for z in range(M):
        l_ref, g_ref = mlp.loss_and_grad(p32[z].astype(np.float64), x[z].astype(np.float64), y[z].astype(np.float64),
                                         n_in, H)
        assert abs(loss[z] - l_ref) <= 1e-5 * abs(l_ref) + 1e-7
        for blk in mlp.unpack(np.arange(g_ref.size), n_in, H):
            ix = np.asarray(blk).ravel()
            assert np.linalg.norm(grad[z][ix] - g_ref[ix]) <= 1e-4 * np.linalg.norm(g_ref[ix]) + 1e-7
    s.close()
