"""Host side of the compressed near field's plans: what the overlap option reserves, and that the reported
shapes are the launched ones."""
import pytest

from test_leaf_form import _plan_data, _random, _uniform


@pytest.fixture(scope="module")
def vp():
    from paper_2501_17967_amd import volpot
    return volpot


def _stages(vp, trees, **kw):
    C, L, off = _plan_data(trees, 1)
    plan = vp.Plan(C, L, host_only=True, tree_offsets=off, **kw)
    out = [{s["name"]: s for s in plan.stages(adj)} for adj in (False, True)]
    plan.close()
    return out


def test_overlap_reserves_units_only_beside_a_chain(vp):
    # host-only plans schedule for 256 compute units of four blocks: overlap 16 is 64 blocks
    trees = [_uniform(7), _random(7, 400, 9)]
    for without, with_ in zip(_stages(vp, trees), _stages(vp, trees, overlap=16)):
        limited = 0
        for n, s in with_.items():
            base = without[n]["n_blocks"]
            if n in ("NEARC48", "ANEARC48"):              # beside the downward chain
                assert base > 960 and s["n_blocks"] == 960, s
            elif n.startswith(("L2L[", "AM2M[")):         # that chain
                assert s["helper"] and s["n_blocks"] == min(base, 64), s
                limited += base > 64
            else:                                         # alone: the whole device
                assert s["n_blocks"] == base, s
        assert limited > 0
