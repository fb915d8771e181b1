"""Device memory of the near-field forms: plans that do not take the compressed form neither build nor hold
its tables, and one that does holds no more than the low-rank form's pair rows took."""
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


def test_compressed_plan_holds_no_more_than_pair_rows():
    from test_leaf_form import _plan_data, _uniform
    from paper_2501_17967_amd import volpot as vp
    C, L, _ = _plan_data([_uniform(9)], 1)
    print("case memory,", len(L), "leaves", flush=True)
    plan = vp.Plan(C, L)
    held = plan.info()["device_bytes"]
    plan.close()
    bound = 4752.9e6   # with two rows of 64 doubles a pair, the scaled input and their schedules
    print("  %d bytes, at most %d" % (held, bound), flush=True)
    assert held <= bound
