"""The strip apply's two launch sequences (the product with E's blocks beside the sweep, from 14 nodes along and
6 across, or after it) on both sides of the line, against the oracle; the bar is that of the other strip tests."""
import numpy as np
import pytest

from oracle import strip
from tests.conftest import rel_max_err
from tests.test_gpu_strip import _run
from workloads import gen

pytestmark = pytest.mark.gpu


@pytest.mark.parametrize("n_panel,q,n_r", [(5, 13, 6), (5, 14, 5), (5, 14, 6), (5, 14, 7), (4, 4, 4), (3, 32, 5),
                                           (3, 32, 6), (6, 13, 24), (6, 14, 24), (3, 16, 32), (3, 12, 32)])
def test_both_sequences_against_the_oracle(device, n_panel, q, n_r):
    import torch

    g, gt = [gen.star_curve(n_panels=n_panel, order=16, scale=s).nodes.reshape(n_panel, 16, 2) for s in (1.0, 0.93)]
    f = lambda p: np.sin(3 * p[:, 0]) * np.exp(p[:, 1]) + 0.5
    sp, v = _run(device, g, gt, f, q, n_r)
    ref, _ = strip.solve(g, gt, f, q=q, n_r=n_r)
    assert rel_max_err(v, ref) < 1e-11
    fv = torch.from_numpy(f(sp.nodes.reshape(-1, 2))).to(device)
    out = torch.full(sp.shape, float("nan"), dtype=torch.float64, device=device)   # every value is written
    sp.apply(fv, out=out)
    assert np.array_equal(out.cpu().numpy(), v)
