"""Which form a structured mesh's steps take, and the forms against each other
where boxes have 512 threads: the launches with the most LDS (about 91 KB with FP64
arithmetic), on several boxes per mesh, in every storage form.  Alone and in a
batch of its own such a mesh takes boxes; beside a 640 x 640 cavity it takes the
march (a periodic channel of at most 16 columns never does: those are planned apart
from the other members, and boxes are always the better there); launch by launch
it takes boxes of one step.  All are equal bit by bit."""
import numpy as np
import pytest

import meshgen

pytestmark = pytest.mark.gpu


@pytest.fixture(scope="module")
def sd():
    import torch
    assert torch.cuda.is_available(), "GPU tests need a HIP device"
    from paper_2007_07347_amd import sdugks
    return sdugks


def _rect(nx, ny):
    mesh = meshgen.structured(meshgen.tanh_nodes(nx), meshgen.tanh_nodes(ny), 0, 0, 1, 0)
    return mesh, [meshgen.bc(meshgen.WALL), meshgen.bc(meshgen.WALL, u=0.1)]


# mesh, and the storage forms in which it takes boxes of 512 threads
WIDE = ("FP64", "FP32NEQ")
SHAPES = [
    (_rect, (301, 120), ("FP64", "FP32DEV", "FP32NEQ")),
    (_rect, (200, 200), ("FP64", "FP32DEV", "FP32NEQ")),
    (_rect, (301, 301), WIDE),
    (meshgen.periodic_box, (210, 200), ("FP64", "FP32DEV", "FP32NEQ")),
    (meshgen.couette, (400, 400), WIDE),
]


@pytest.mark.parametrize("prec", ["FP64", "FP32DEV", "FP32NEQ"])
@pytest.mark.parametrize("scheme,macro", [(0, 1), (0, 0), (1, 1)])
def test_boxes_of_512_threads(sd, prec, scheme, macro):
    kw = dict(cfl=0.5 if macro else 0.1, precision=getattr(sd, prec), macro=macro, scheme=scheme)

    def make(mesh, bcs, seed):
        s = sd.Solver(mesh, bcs, nu=4e-3 if macro else 2e-2, **kw)
        f, W, G = meshgen.random_state(s.n_cells, seed=seed, amp=0.02)
        if macro:
            G[:] = 0.0
        s.set_state(f, W, G)
        return s

    chosen = [(mk, n) for mk, n, precs in SHAPES if prec in precs]
    problems = [mk(*n) for mk, n in chosen]
    alone, eager, single, beside = ([make(*p, k) for k, p in enumerate(problems)] for _ in range(4))
    big = make(*meshgen.cavity(640), 99)
    b = sd.Batch(beside + [big])
    b.step(22)
    b.step(1)
    for k, (_, n) in enumerate(chosen):
        print(prec, scheme, macro, n, alone[k].schedule(), b.schedule(k), flush=True)
        assert alone[k].schedule()["form"] == "boxes" and alone[k].schedule()["threads"] == 512
        assert alone[k].schedule()["groups"] > 1
        assert b.schedule(k)["form"] == "march"
        one = sd.Batch([single[k]])
        assert one.schedule(0) == alone[k].schedule()
        one.step(22)
        one.step(1)
        one.close()
        alone[k].step(23)
        eager[k].step_eager(23)
        x = alone[k].state()
        assert all(np.isfinite(v).all() for v in x)
        for other in (eager[k], single[k], beside[k]):
            assert all(np.array_equal(v, w) for v, w in zip(x, other.state())), n
    b.close()
    for s in alone + eager + single + beside + [big]:
        s.close()


def test_schedules_of_the_other_forms(sd):
    """Tiles, the two-kernel step and whole meshes in one box; refused calls."""
    mesh, bcs = meshgen.cavity(40)
    s = sd.Solver(mesh, bcs, nu=1e-3, structured=1, tile_cells=32, block_threads=128)
    assert s.schedule() == {"form": "tiles", "threads": 128, "steps": 1, "groups": 50}
    t = sd.Solver(mesh, bcs, nu=1e-3, tile_cells=-1)
    assert t.schedule()["form"] == "two-kernel"
    w = sd.Solver(*meshgen.couette(4, 32), nu=1e-2)
    assert w.schedule() == {"form": "boxes", "threads": 128, "steps": 1000, "groups": 1}
    b = sd.Batch([s, w])
    assert b.schedule(0)["form"] == "tiles" and b.schedule(1)["form"] == "boxes"
    for k in (-1, 2):
        with pytest.raises(sd.SdugksError):
            b.schedule(k)
    b.close()
    for x in (s, t, w):
        x.close()


@pytest.mark.parametrize("prec", ["FP64", "FP32DEV", "FP32NEQ"])
def test_threads_asked_for_are_launched(sd, prec):
    """Explicit schedules of the general step run on the threads they name.  On more
    tiles than the chip takes at once (785 of 64 cells, 1569 of 32 and 3138 of 16 here:
    an odd last tile among them) a workgroup has two tiles; bits as with one tile
    per workgroup, alone and in a batch beside a smaller mesh of other pitches."""
    mesh, bcs = meshgen.cylinder_ogrid(251, 100, seed=6)
    small = meshgen.cylinder_ogrid(40, 12, seed=7, quad_layers=12)
    ex = np.array([0, 1, 0, -1, 0, 1, -1, -1, 1.0])
    ey = np.array([0, 0, 1, 0, -1, 1, 1, -1, -1.0])

    def make(mesh, bcs, sched, seed):
        s = sd.Solver(mesh, bcs, nu=4e-3, cfl=0.4, precision=getattr(sd, prec), **sched)
        f, _, _ = meshgen.random_state(s.n_cells, seed=seed, amp=0.02)
        s.set_state(f, np.c_[f.sum(1), f @ ex, f @ ey])
        return s

    refs = []
    for m, seed in (((mesh, bcs), 3), (small, 4)):
        s = make(*m, dict(tile_cells=16, block_threads=64), seed)
        s.step(7)
        refs.append(s.state())
        s.close()
    for tc, bt, tiles in ((64, 256, 2), (32, 256, 2), (16, 256, 2), (32, 128, 2), (16, 128, 2), (16, 64, 1)):
        sched = dict(tile_cells=tc, block_threads=bt)
        s = make(mesh, bcs, sched, 3)
        v = s.schedule()
        n = sd.tiling(mesh, bcs, nu=4e-3, cfl=0.4, precision=getattr(sd, prec), **sched)["n_tiles"]
        print(prec, tc, bt, n, v, flush=True)
        assert v["form"] == "tiles" and v["threads"] == bt and v["groups"] == -(-n // tiles)
        s.step(7)
        members = [make(*small, sched, 4), make(mesh, bcs, sched, 3), make(*small, sched, 4)]
        b = sd.Batch(members)
        assert b.schedule(1)["threads"] == bt
        b.step(7)
        for x, ref in zip((s, *members), (refs[0], refs[1], refs[0], refs[1])):
            assert all(np.array_equal(p, q) for p, q in zip(x.state(), ref)), (tc, bt)
            assert np.isfinite(x.state()[0]).all()
        b.close()
        for x in (s, *members):
            x.close()


@pytest.mark.parametrize("prec", ["FP64", "FP32DEV"])
def test_odd_steps_do_not_plan_again(sd, prec):
    """An odd number of batched steps, or of a member's launches alone (a mesh in one
    box takes any number of steps in one), changes the buffers that members read.
    The batch keeps its tables; states are those of the members stepped alone, and
    the batch works on after a change of members with odd indices."""
    meshes = [meshgen.couette(4, 32), meshgen.cavity(48), meshgen.cylinder_ogrid(40, 12, seed=2), meshgen.couette(6, 20)]

    def make(k):
        s = sd.Solver(*meshes[k], nu=4e-3, cfl=0.5, precision=getattr(sd, prec))
        f, W, _ = meshgen.random_state(s.n_cells, seed=k, amp=0.02)
        s.set_state(f, W)
        return s

    alone, members = [make(k) for k in range(4)], [make(k) for k in range(4)]
    b = sd.Batch(members)
    assert b.builds() == 1
    total = [0] * 4
    for n, stepped in ((1, ()), (3, (0,)), (2, (0, 1)), (5, (2, 3)), (1, (0, 1, 2)), (4, ())):
        for k in stepped:
            members[k].step(4)
            total[k] += 4
        b.step(n)
        total = [t + n for t in total]
    assert b.builds() == 1
    b.set_members(members[1:])
    assert b.builds() == 2
    b.step(3)
    total = [total[0]] + [t + 3 for t in total[1:]]
    assert b.builds() == 2
    for s, m, n in zip(alone, members, total):
        s.step(n)
        assert m.info()["step"] == n
        assert all(np.array_equal(x, y) for x, y in zip(s.state(), m.state()))
    b.debug_fail_next_build()
    with pytest.raises(sd.SdugksError):
        b.step(1)
    with pytest.raises(sd.SdugksError):
        b.step(2)
    b.set_members(members)
    b.step(1)
    b.close()
    for s in alone + members:
        s.close()


def test_profiled_steps_are_launched_as_steps_are(sd):
    """A mesh in one box takes all profiled steps in one launch, as sdugks_step does,
    and its time is per step: well below that of launches of one step each (2.2
    against 5 us and more)."""
    s = sd.Solver(*meshgen.couette(4, 32), nu=1e-2)
    s.step_profiled(50)
    together = min(s.step_profiled(400)["k_step_cart"] for _ in range(3))
    each = min(s.step_profiled(1)["k_step_cart"] for _ in range(50))
    assert s.info()["step"] == 50 + 3 * 400 + 50
    s.close()
    print(together, each, flush=True)
    assert together < 0.75 * each


def test_autotuner_reports_the_threads_that_ran(sd):
    """Every candidate runs on the threads it names; the library's choice (0) is
    reported as what it is, and where that is the launch of another candidate
    (up to 768 tiles: 256 threads) both have the one time."""
    from paper_2007_07347_amd import autotune
    mesh, bcs = meshgen.cylinder_ogrid(60, 20, seed=1)
    best, table = autotune.autotune(mesh, bcs, steps=20, cache=None, nu=2e-3, cfl=0.5)
    rows = {(r["tile_cells"], r["block_threads"]): r for r in table}
    assert set(rows) == set(autotune.CANDIDATES)
    assert all(r["threads"] == bt for (_, bt), r in rows.items() if bt)
    assert rows[64, 0]["threads"] == 256 and rows[64, 0]["ms"] == rows[64, 256]["ms"]
    assert set(best) == {"tile_cells", "block_threads", "structured"}
