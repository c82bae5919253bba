"""The two forms of the structured step -- waves marching along strips, and
boxes that take several steps per launch -- at the sizes where their cuts can
go wrong: meshes that just fit a box or are one cell too large, halves and
remainders of strips (60 columns, or multiples of eight) and boxes (16 and 32 cells), periodic meshes
narrower than a box (rows that wrap inside it) and wider ones, two cells along
an axis.  Small meshes alone take boxes; in one batch with a 640 x 640 cavity
they take the march; one launch per step (step_eager) takes boxes of one step.
(Periodic meshes of at most 16 columns are planned apart from the others there
and take boxes in the batch too.)
All use the same arithmetic in the same order, so the results are equal bit by
bit."""
import sys

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


def _half_channel(nx, ny):
    mesh = meshgen.structured(np.linspace(0.0, 1.0, nx + 1), meshgen.tanh_nodes(ny, 1.0), tag_bottom=3, tag_right=1,
                              tag_top=0, tag_left=2)
    return mesh, [meshgen.bc(meshgen.WALL), meshgen.bc(meshgen.OUTLET), meshgen.bc(meshgen.INLET, u=0.05),
                  meshgen.bc(meshgen.SYMMETRY)]


def _walls_x(nx, ny):
    """Walls left and right (the right one moving), periodic in y."""
    mesh = meshgen.structured(meshgen.tanh_nodes(nx, 1.2), np.linspace(0.0, 0.5, ny + 1), tag_bottom=0, tag_right=2,
                              tag_top=1, tag_left=3)
    return mesh, [meshgen.bc(meshgen.PERIODIC, partner=1, shift=(0.0, 0.5)),
                  meshgen.bc(meshgen.PERIODIC, partner=0, shift=(0.0, -0.5)),
                  meshgen.bc(meshgen.WALL, v=0.05), meshgen.bc(meshgen.WALL)]


def _rect(nx, ny):
    mesh = meshgen.structured(meshgen.tanh_nodes(nx), meshgen.tanh_nodes(ny), 0, 0, 1, 0)
    return mesh, [meshgen.bc(meshgen.WALL), meshgen.bc(meshgen.WALL, u=0.1)]


SHAPES = {
    "walls": (_rect, [(2, 2), (2, 9), (9, 2), (14, 16), (14, 32), (15, 33), (30, 16), (31, 17), (60, 5), (61, 60), (62, 8),
                      (63, 24), (104, 17), (112, 9), (120, 31), (121, 64), (168, 33), (181, 90)]),
    "periodic": (meshgen.periodic_box, [(2, 2), (4, 64), (5, 65), (16, 32), (17, 33), (64, 8), (65, 9), (61, 120), (104, 9)]),
    "periodic_x": (meshgen.couette, [(2, 3), (4, 32), (4, 128), (4, 129), (17, 8), (65, 20)]),
    "periodic_y": (_walls_x, [(2, 2), (9, 20), (30, 16), (61, 32)]),
    "open": (_half_channel, [(13, 7), (31, 15), (62, 40), (104, 18)]),
}
CASES = [(kind, n) for kind, (_, sizes) in SHAPES.items() for n in sizes]


@pytest.mark.parametrize("prec", ["f64", "fp32dev", "fp32neq"])
@pytest.mark.parametrize("scheme,macro", [(0, 1), (0, 0), (1, 1)])
def test_forms_are_equal_bit_by_bit(sd, prec, scheme, macro):
    """Generic states advanced 23 steps (a count that is no multiple of a
    launch's steps, nor of a graph's): alone, in the batch, and launch by
    launch, all equal."""
    p = {"f64": sd.FP64, "fp32dev": sd.FP32DEV, "fp32neq": sd.FP32NEQ}[prec]
    kw = dict(cfl=0.5 if macro else 0.1, precision=p, macro=macro, scheme=scheme)

    def make(mesh, bcs, nu, seed):
        s = sd.Solver(mesh, bcs, nu=nu, **kw)
        f, W, G = meshgen.random_state(s.n_cells, seed=seed, amp=0.02)
        if macro:
            G[:] = 0.0
        s.set_state(f, W, G)
        return s

    problems = [(*SHAPES[kind][0](*n), 4e-3 if macro else 2e-2) for kind, n in CASES]
    alone, eager, batched = ([make(*pr, k) for k, pr in enumerate(problems)] for _ in range(3))
    big = make(*meshgen.cavity(640), 1e-3, 99)
    b = sd.Batch(batched + [big])
    b.step(22)
    b.step(1)
    for (kind, n), x, y, z in zip(CASES, alone, eager, batched):
        print(prec, scheme, macro, kind, n, flush=True)
        x.step(23)
        y.step_eager(23)
        sx, sy, sz = x.state(), y.state(), z.state()
        assert all(np.isfinite(v).all() for v in sx)
        for v, w, u in zip(sx, sy, sz):
            assert np.array_equal(v, w) and np.array_equal(v, u), (kind, n)
    b.close()
    for s in alone + eager + batched + [big]:
        s.close()
    sys.stdout.flush()
