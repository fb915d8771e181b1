"""Both forms of the near field over the options that cut, share and reorder their launches: the low-rank form
(trees below 512 leaves) on a graded tree of 460 leaves, and the compressed form on forests with leaves
above level 2. The form is read from the plan, so that a change of the threshold cannot redirect a test.

Tolerance 1e-13 of the output's norm against the dense tables of the same plan (sums in another order and
tables equal to 1e-14 of the self table's norm); bitwise where only launches differ.
"""
import ctypes

import numpy as np
import pytest

from test_leaf_form import _plan_data, _random, _uniform, rel

pytestmark = pytest.mark.gpu
ORDERS = [0.0, 1e-11, 1e-9, 1e-6]


@pytest.fixture(scope="module")
def vp():
    from paper_2501_17967_amd import volpot
    return volpot


def _form(plan):
    s = plan.stages()[-1]
    assert s["name"] == "NEAR+LOCT"
    return "low-rank" if s["inner"] == 64 else "compressed"


def _values(n, seed, k=3):
    import torch
    rng = np.random.default_rng(seed)
    return [torch.from_numpy(rng.standard_normal((n, 256))).cuda() for _ in range(k)]


def _dense(vp, C, L, off, eps, x):
    plan = vp.Plan(C, L, tree_offsets=off, eps=eps, dense_near=True, dense_m2l=True)
    out = [(plan.apply(v).cpu().numpy(), plan.apply_adjoint(v).cpu().numpy()) for v in x]
    plan.close()
    return out


GRADED = lambda: _plan_data([_random(9, 60, 8)], 6)


@pytest.fixture(scope="module")
def graded(vp):
    C, L, off = GRADED()
    x = _values(len(L), 6)
    return C, L, off, x, {eps: _dense(vp, C, L, off, eps, x) for eps in (0.0, 1e-6)}


@pytest.mark.parametrize("eps", [0.0, 1e-6])
@pytest.mark.parametrize("kw", [{}, {"overlap": 16}, {"split_min": 1}, {"split_min": 3}, {"split_min": -1},
                                {"deterministic": True}, {"tile_leaf": 32}, {"tile_leaf": 64}, {"tile_box": 32},
                                {"tile_leaf": 64, "tile_box": 64, "split_min": 1, "overlap": 32}],
                         ids=lambda kw: "-".join("%s=%s" % i for i in kw.items()) or "default")
def test_low_rank_form_matches_dense_tables(vp, graded, kw, eps):
    import torch
    C, L, off, x, want = graded
    print("case low-rank", kw, "eps", eps, len(L), "leaves", flush=True)
    eager = vp.Plan(C, L, eps=eps, **kw)
    graph = vp.Plan(C, L, eps=eps, use_graph=True, **kw)
    assert _form(eager) == _form(graph) == "low-rank"
    buf, u, b = torch.empty_like(x[0]), torch.empty_like(x[0]), torch.empty_like(x[0])
    for v, (uw, bw) in zip(x, want[eps]):   # the second and third pass replay the graphs on new values
        e = (eager.apply(v), eager.apply_adjoint(v))
        buf.copy_(v)
        graph.apply(buf, out=u)
        graph.apply_adjoint(buf, out=b)
        torch.cuda.synchronize()
        assert torch.equal(e[0], u) and torch.equal(e[1], b)
        assert rel(u.cpu().numpy(), uw) <= 1e-13 and rel(b.cpu().numpy(), bw) <= 1e-13
    eager.close()
    graph.close()


SHALLOW = {
    "roots": lambda: [_uniform(0)] * 600,                                     # no box below level 0
    "level-1": lambda: [_uniform(1)] * 140,                                   # near field only
    "mixed": lambda: [_uniform(0)] * 5 + [_random(3, 30, 6), _uniform(1), _uniform(4), _uniform(0), _random(4, 25, 7)],
    "level-1-leaves": lambda: [_quarter()] * 3 + [_uniform(4), _uniform(4)],   # with W and X lists
}


def _quarter():
    # three leaves of level 1, as near to refined boxes as 2:1 balance lets them lie
    from workloads import gen
    leaves = {(1, 0, 1), (1, 1, 0), (1, 1, 1), (2, 0, 1), (2, 1, 0), (2, 1, 1), (3, 1, 0), (3, 0, 1), (3, 1, 1)}
    leaves |= {(4, x, y) for x in (0, 1) for y in (0, 1)}
    assert gen.balance(set(leaves)) == leaves
    return leaves


@pytest.mark.parametrize("kw", [{}, {"overlap": 16}, {"split_min": 1}, {"deterministic": True}],
                         ids=lambda kw: "-".join("%s=%s" % i for i in kw.items()) or "default")
@pytest.mark.parametrize("name", sorted(SHALLOW))
def test_compressed_form_with_leaves_above_level_2(vp, name, kw):
    trees = SHALLOW[name]()
    C, L, off = _plan_data(trees, 7)
    print("case", name, kw, len(L), "leaves,", len(trees), "trees", flush=True)
    assert L.min() < 2
    x = _values(len(L), 7, 1)
    plan = vp.Plan(C, L, tree_offsets=off, **kw)
    assert _form(plan) == "compressed"
    (u, b), = _dense(vp, C, L, off, 0.0, x)
    for _ in range(2):
        assert rel(plan.apply(x[0]).cpu().numpy(), u) <= 1e-13
        assert rel(plan.apply_adjoint(x[0]).cpu().numpy(), b) <= 1e-13
    plan.close()


def _launches(vp, plan, x):
    # kernels of one forward and one adjoint apply, counted in captured graphs
    import torch
    hip = ctypes.CDLL(vp.lib()._name)   # the runtime's own functions, found through the library
    out = torch.empty_like(x)
    s = torch.cuda.Stream()
    n = []
    for fn in (plan.apply, plan.apply_adjoint):
        torch.cuda.synchronize()
        graph, nodes = ctypes.c_void_p(), ctypes.c_size_t()
        assert hip.hipStreamBeginCapture(ctypes.c_void_p(s.cuda_stream), 1) == 0   # 1: this thread's calls only
        fn(x, out=out, stream=s)
        assert hip.hipStreamEndCapture(ctypes.c_void_p(s.cuda_stream), ctypes.byref(graph)) == 0
        assert hip.hipGraphGetNodes(graph, None, ctypes.byref(nodes)) == 0
        n.append(nodes.value)
        assert hip.hipGraphDestroy(graph) == 0
    return n


@pytest.mark.parametrize("eps", ORDERS)
@pytest.mark.parametrize("name,trees,saved", [
    ("uniform-64", [_uniform(3)], (2, 2)),          # S2M and the two pair stages, and their transposes
    ("graded-460", [_random(9, 60, 8)], (2, 2)),
    ("uniform-1024", [_uniform(5)], (1, 0)),        # edge and corner stage
    ("graded-1360", [_random(200, 200, 8)], (1, 0)),
    ("uniform-4096", [_uniform(6)], (0, 0)),        # too large to share a launch
])
def test_small_stages_share_launches(vp, name, trees, saved, eps):
    C, L, off = _plan_data(trees, 3)
    print("case launches", name, "eps", eps, flush=True)
    plan = vp.Plan(C, L, eps=eps)
    x, = _values(len(L), 3, 1)
    plan.apply(x), plan.apply_adjoint(x)
    stages = [sum(s["n_tiles"] > 0 for s in plan.stages(adj)) for adj in (False, True)]
    stages[0] += _form(plan) == "low-rank"          # the scaled input
    got = _launches(vp, plan, x)
    print("  stages", stages, "launches", got, flush=True)
    assert (stages[0] - got[0], stages[1] - got[1]) == saved
    plan.close()


@pytest.mark.parametrize("name,trees", [
    ("low-rank", [_random(9, 30, 8), _uniform(2), _uniform(0), _random(4, 25, 7)]),
    ("compressed", [_random(3, 60, 7), _uniform(4), _uniform(0), _random(5, 40, 9)]),
    ("compressed", [_uniform(7), _random(5, 400, 10), _uniform(1)]),
])
def test_nan_stays_in_its_tree_and_its_apply(vp, name, trees):
    # a NaN in one tree of a forest reaches no other tree, and nothing of it is left in the plan's memory
    import torch
    C, L, off = _plan_data(trees, 8)
    print("case NaN", name, len(L), "leaves", flush=True)
    plan = vp.Plan(C, L, tree_offsets=off)
    assert _form(plan) == name
    x, = _values(len(L), 8, 1)
    for fn in (plan.apply, plan.apply_adjoint):
        clean = fn(x).clone()
        for t in range(len(trees)):
            bad = x.clone()
            bad[off[t] + (off[t + 1] - off[t]) // 2, 77] = float("nan")
            got = fn(bad)
            other = torch.ones(len(L), dtype=torch.bool, device="cuda")
            other[off[t]:off[t + 1]] = False
            assert torch.equal(got[other], clean[other]) and bool(torch.isnan(got[~other]).all())
            assert torch.equal(fn(x), clean)
    plan.close()
