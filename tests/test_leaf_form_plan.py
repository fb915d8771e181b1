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


@pytest.mark.parametrize("trees,tile", [([_uniform(5)], 16), ([_random(3, 260, 9)], 16), ([_uniform(7)], 32)])
def test_leaf_output_reports_the_tiles_it_launches(vp, trees, tile):
    n = sum(len(t) for t in trees)
    assert (n <= 8192) == (tile == 16)
    for split_min in (0, 1, -1):
        for st, name in zip(_stages(vp, trees, split_min=split_min), ("NEAR+LOCT", "ANEAR+ALOCT")):
            s = st[name]
            assert s["tile"] == tile and s["n_tiles"] == -(-n // tile), s
            assert s["flops_issued"] == 2.0 * 256 * s["inner"] * tile * s["n_tiles"]
            assert split_min >= 0 or s["n_blocks"] == s["n_tiles"], s


def test_leaves_without_neighbours_are_no_targets(vp):
    # trees of one leaf receive and send nothing; beside others they add nothing to the edge and corner stages
    fwd, adj = _stages(vp, [_uniform(0)] * 600)
    assert [n for n in fwd if fwd[n]["n_tiles"]] == ["S2M", "NEAR+LOCT"]
    assert "ANEARC" not in adj and "ANEARC48" not in adj
    trees = [_random(3, 260, 9)]
    for alone, beside in zip(_stages(vp, trees), _stages(vp, [_uniform(0)] * 40 + trees)):
        for n in alone:
            if n in ("NEARC", "NEARC48", "ANEARC", "ANEARC48"):
                assert beside[n]["n_tiles"] == alone[n]["n_tiles"], n
