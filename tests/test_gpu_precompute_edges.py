"""Precompute at the edges of its row slices and tiles, in every precision,
against numpy in 64 bits with componentwise rounding bounds."""
import math

import numpy as np
import pytest

import synth
from tests.gpu_util import have_gpu

pytestmark = [pytest.mark.gpu, pytest.mark.skipif(not have_gpu(), reason="no GPU")]

# one row and column; around 32 and 64 rows; one past a tile; many slices of few
# tiles; 10 and 11 tile rows (either side of the rule for few tiles); an odd and
# an even number of tile rows
SHAPES = [(1, 1), (31, 5), (33, 64), (64, 65), (65, 130), (1500, 64), (700, 640), (700, 641), (300, 190), (520, 257)]


@pytest.mark.parametrize("prec", ["fp64", "fp32", "bf16x3", "bf16x2"])
@pytest.mark.parametrize("m,n", SHAPES)
def test_products(m, n, prec):
    import paper_2501_12928_amd as eor
    inst = synth.small(seed=m + n, m=m, n=n, n_k=1, n_theta=1)
    W = inst.T / np.sqrt(inst.noise_var)[:, None]
    A = W.conj().T @ W
    mag = np.abs(W).T @ np.abs(W)
    wd = inst.d / np.sqrt(inst.noise_var)
    dbar = W.conj().T @ wd
    # FP32: 64-row partial sums of rounded products; two-term bf16 drops 2^-16 per product and part
    eps = {"fp64": (m + 8) * 2.0 ** -52, "fp32": 160 * 2.0 ** -24, "bf16x3": 160 * 2.0 ** -24,
           "bf16x2": 160 * 2.0 ** -24 + 2.0 ** -13}[prec]
    print(f"gpu: precompute {m} x {n} {prec}", flush=True)
    ctx = eor.Context(0).precompute(inst.T, inst.noise_var, inst.d, 1, inst.bin_of, inst.fixed_var, prec=prec)
    gA, gd, c, K0 = ctx.export_precompute()
    ctx.close()
    assert np.all(np.abs(gA.cpu().numpy() - A) <= eps * mag)
    assert np.all(np.abs(gd.cpu().numpy() - dbar) <= (m + 8) * 2.0 ** -52 * (np.abs(W).T @ np.abs(wd)))
    cr = float(np.sum(np.abs(wd) ** 2))
    assert abs(c - cr) <= (m + 8) * 2.0 ** -52 * cr
    ref = -m * math.log(math.pi) - float(np.sum(np.log(inst.noise_var)))
    assert abs(K0 - ref) <= (m + 8) * 2.0 ** -52 * (m * math.log(math.pi) + float(np.sum(np.abs(np.log(inst.noise_var)))))
