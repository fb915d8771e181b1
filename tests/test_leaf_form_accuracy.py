"""Accuracy of the compressed near field where its bases carry what lies beyond an adjacent box: W-list
boxes in all directions, refined further than a leaf's own polynomial resolves.

One tree per W offset off the diagonals: a target leaf of level 4 and, in the W box there, a leaf of
level 8 at the box's far corner beside the line through the target's own edge. The field of that leaf alone
is compared, leaf by leaf, with the plan that applies the dense tables; both share the far field.

Tolerance 1e-14 of the field at each leaf: the bases leave 2e-15 of the field of a point charge anywhere
in a W box, the multipole reaches that box in four sums and the target in one more, 1e-15 each.
"""
import numpy as np
import pytest

from test_leaf_form import _plan_data, _uniform
from workloads import gen

OFFSETS = [(sx * a, sy * b) for a, b in ((1, 3), (3, 1)) for sx in (1, -1) for sy in (1, -1)]
TARGET = (4, 7, 7)
SOURCE_LEVEL = 8
TOL = 1e-14


def _tree(corner):
    # leaves, and the one of SOURCE_LEVEL inside the W box whose far corner is at the given distance from
    # the target's centre (in its half-widths)
    n = 1 << SOURCE_LEVEL
    s = n // 16 // 2                        # the target's half-width in units of the finest leaves
    at = [(2 * TARGET[1 + k] + 1) * s + corner[k] * s for k in (0, 1)]
    # the corner is the box's far one in the larger coordinate and its near one in the other
    big = 0 if abs(corner[0]) > abs(corner[1]) else 1
    key = [at[k] - 1 if (corner[k] > 0) == (k == big) else at[k] for k in (0, 1)]
    leaves = _uniform(4)
    for l in range(4, SOURCE_LEVEL):
        k = (l, key[0] >> (SOURCE_LEVEL - l), key[1] >> (SOURCE_LEVEL - l))
        leaves.remove(k)
        leaves |= {(l + 1, 2 * k[1] + a, 2 * k[2] + b) for a in (0, 1) for b in (0, 1)}
    leaves = gen.balance(leaves)
    source = (SOURCE_LEVEL, key[0], key[1])
    assert TARGET in leaves and source in leaves
    return leaves, source


def _forest():
    trees, sources = zip(*[_tree(c) for c in OFFSETS])
    C, L, off = _plan_data(trees, 4)

    def index(t, k):
        h = 1.0 / (1 << k[0])
        c = np.array([-1 + (2 * k[1] + 1) * h, -1 + (2 * k[2] + 1) * h])
        i = [i for i in range(off[t], off[t + 1]) if L[i] == k[0] and np.all(np.abs(C[i] - c) < 1e-12)]
        assert len(i) == 1
        return i[0]
    return C, L, off, [index(t, TARGET) for t in range(len(trees))], [index(t, s) for t, s in enumerate(sources)]


def test_sources_lie_in_w_boxes_off_the_diagonals():
    C, L, off, target, source = _forest()
    assert len(L) >= 512
    for t, c in enumerate(OFFSETS):
        d = (C[source[t]] - C[target[t]]) * 16   # in the target's half-widths
        w = (np.floor(d) + 0.5)                  # centre of the box of half the target's size around it
        assert sorted(np.abs(w)) == [1.5, 2.5] and np.array_equal(np.sign(w), np.sign(c))


@pytest.mark.gpu
def test_fields_of_w_boxes_keep_their_digits():
    import torch
    from paper_2501_17967_amd import volpot as vp
    C, L, off, target, source = _forest()
    print("case W boxes,", len(L), "leaves", flush=True)
    plans = [vp.Plan(C, L, tree_offsets=off, dense_near=d) for d in (False, True)]
    f = np.zeros((len(L), 256))
    f[source] = 4.0 ** SOURCE_LEVEL
    u, ref = [p.apply(torch.from_numpy(f).cuda()).cpu().numpy() for p in plans]
    for t in range(len(OFFSETS)):
        near = [i for i in range(off[t], off[t + 1]) if np.max(np.abs(C[i] - C[source[t]])) < 0.25]
        e = {i: np.max(np.abs(u[i] - ref[i])) / np.max(np.abs(ref[i])) for i in near}
        print("  offset", OFFSETS[t], "target %.1e" % e[target[t]], "largest %.1e" % max(e.values()), flush=True)
        assert max(e.values()) <= TOL, OFFSETS[t]
    # a unit cotangent at each node of the row (column) that faces the box
    for n in range(16):
        g = np.zeros((len(L), 16, 16))
        for t, c in enumerate(OFFSETS):
            j, i = (n, 15 if c[0] > 0 else 0) if abs(c[0]) > abs(c[1]) else (15 if c[1] > 0 else 0, n)
            g[target[t], j, i] = 1.0
        g = torch.from_numpy(g.reshape(len(L), 256)).cuda()
        b, ref = [p.apply_adjoint(g).cpu().numpy() for p in plans]
        e = [np.max(np.abs(b[s] - ref[s])) / np.max(np.abs(ref[s])) for s in source]
        print("  node", n, "adjoint %.1e" % max(e), flush=True)
        assert max(e) <= TOL, (n, e)
    for p in plans:
        p.close()


@pytest.mark.gpu
def test_values_near_the_largest_number():
    # s^2 f lies far inside the type's range, and at this level so does what the translations make of it;
    # powers of two change no digit
    import torch
    from paper_2501_17967_amd import volpot as vp
    C, L, off = _plan_data([_uniform(7)], 5)
    print("case large values,", len(L), "leaves", flush=True)
    g = np.random.default_rng(5).uniform(-1.0, 1.0, (len(L), 256))   # of both signs: the total charge stays in range too
    f = torch.from_numpy(g).cuda() * 2.0 ** 1023
    plan = vp.Plan(C, L)
    u, small = plan.apply(f), plan.apply(f * 2.0 ** -60)
    assert bool(torch.isfinite(u).all()) and torch.equal(u, small * 2.0 ** 60)
    plan.close()
