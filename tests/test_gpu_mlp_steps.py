"""GPU test of the MLP's products where the reduction's steps of 16 do not fill
the groups that are loaded together: weight products over 32 rows upwards, in
one slice and in several of an odd number of steps."""
import numpy as np
import pytest
import torch

import oracle
from test_gpu_mlp import DEV, TOL, inputs, run_oracle, targets, to_bits, weights

pytestmark = pytest.mark.gpu


@pytest.mark.parametrize("n", [32, 96, 1025, 1584, 4100])
def test_gradients(n):
    from paper_2604_01844_amd.mlp import InitMLP
    w = weights(3)
    x, rows = inputs(n, 11)
    t = targets(n, 12)
    net = InitMLP(w, DEV)
    xb = torch.from_numpy(to_bits(x)).to(DEV)
    acts = net.forward(xb, rows, keep_transposes=True)
    _, _, dz3, dz3t = net.heads(acts, n, torch.from_numpy(t.astype(np.float32)).to(DEV))
    g = net.backward(xb.t().contiguous(), rows, acts, dz3, dz3t)
    ref = run_oracle(x, w, t.astype(np.float32).astype(np.float64), n)[4]
    for k in ("dw1", "db1", "dw2", "db2", "dw3", "db3"):
        assert oracle.rel_l2(g[k].cpu().numpy(), ref[k]) <= TOL, k  # the bar of the other sizes
