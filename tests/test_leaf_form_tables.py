"""Plans that do not take the compressed near field neither build nor hold its tables."""
import numpy as np
import pytest

pytestmark = pytest.mark.gpu


@pytest.mark.parametrize("eps,ne", [(0.0, 80), (1e-6, 32)])
def test_small_plan_holds_no_compressed_tables(eps, ne):
    from paper_2501_17967_amd import volpot as vp
    C = np.array([[x, y] for x in (-0.5, 0.5) for y in (-0.5, 0.5)])
    print("case four leaves, eps", eps, flush=True)
    plan = vp.Plan(C, np.full(4, 1, dtype=np.int32), eps=eps)
    # every other table, each with its transpose: 33 adjacent relations with rank-64 factors at most, the
    # self table's slices, maps between leaf values and expansions (2 + 40), translations (40 one- and
    # two-level, 40 M2L), and 1 MiB for the core, the diagonals, descriptors and the plan itself
    doubles = 33 * 256 * 256 + 64 * 256 * 64 + 4 * 256 * 64 + 42 * 256 * ne + 80 * ne * ne
    held = plan.info()["device_bytes"]
    print("  %d bytes, at most %d" % (held, 16 * doubles + (1 << 20)), flush=True)
    assert held <= 16 * doubles + (1 << 20)
    plan.close()
