"""The autotuner starts from the library's own defaults, can return them, and does not take shapes that were
timed for earlier kernels."""
import numpy as np
import pytest

from workloads import gen

pytestmark = pytest.mark.gpu


@pytest.fixture(scope="module")
def vp():
    from paper_2501_17967_amd import volpot
    return volpot


def _key(w, version, ne=80):
    # the signature of a single tree's cache lines: FNV-1a over the version, the number of trees, leaves per
    # level, sizes, reals per expansion, forms and device
    import torch
    prop = torch.cuda.get_device_properties(0)
    h = 1469598103934665603
    vals = [version, 1] + np.bincount(w.levels, minlength=32).tolist() + [len(w.levels), ne, 0, 0]
    vals += list(prop.gcnArchName.encode()) + [prop.multi_processor_count]
    for v in vals:
        for b in range(8):
            h = ((h ^ ((int(v) >> (8 * b)) & 0xff)) * 1099511628211) % (1 << 64)
    return "%016x" % h


def test_defaults_can_be_remembered_and_old_shapes_are_not_taken(vp, tmp_path):
    w = gen.config1(0)
    print("case autotune cache,", w.n_leaves, "leaves", flush=True)
    cache = tmp_path / "tune.txt"
    cache.write_text("%s 64 64 1 16 64 16 0.001\n" % _key(w, 3))   # timed before the present defaults
    best, ms = vp.autotune(w.centres, w.levels, cache=str(cache))
    assert ms > 0.001
    lines = cache.read_text().splitlines()
    assert len(lines) == 2 and lines[1].split()[0] == _key(w, 4)
    for tile_leaf, tile_box in ((16, 16), (16, 0), (32, 0)):       # the defaults are valid lines
        cache.write_text("%s %d %d 0 0 16 32 0.5\n" % (_key(w, 4), tile_leaf, tile_box))
        got, ms = vp.autotune(w.centres, w.levels, cache=str(cache))
        assert ms == 0.5 and (got["tile_leaf"], got["tile_box"]) == (tile_leaf, tile_box)


@pytest.mark.parametrize("name", ["config1", "config2"])
def test_tuned_plan_is_not_slower_than_the_default(vp, name):
    import torch
    w = getattr(gen, name)(0)
    print("case autotune", name, w.n_leaves, "leaves", flush=True)
    best, _ = vp.autotune(w.centres, w.levels)
    plans = [vp.Plan(w.centres, w.levels), vp.Plan(w.centres, w.levels, **best)]
    f = torch.from_numpy(w.f).cuda()
    u, b = torch.empty_like(f), torch.empty_like(f)
    t = [[], []]
    for rep in range(60):
        for k, p in enumerate(plans):
            e = [torch.cuda.Event(enable_timing=True) for _ in range(2)]
            e[0].record()
            for _ in range(5):
                p.apply(f, out=u)
                p.apply_adjoint(f, out=b)
            e[1].record()
            torch.cuda.synchronize()
            t[k].append(e[0].elapsed_time(e[1]))
    d, s = [float(np.median(x[10:])) / 5 * 1e3 for x in t]
    print("  default %.1f us, tuned %s %.1f us" % (d, best, s), flush=True)
    assert s <= 1.05 * d    # a candidate replaces the defaults only where it measured 1.5% faster
    for p in plans:
        p.close()
