"""Rounding of the steps' building blocks: the reciprocal of a density is that
of an FP64 division, the reconstruction takes one offset from a cell's centre to
the foot point."""
import numpy as np
import pytest

import meshgen

pytestmark = pytest.mark.gpu

EX = np.array([0, 1, 0, -1, 0, 1, -1, -1, 1], dtype=float)
EY = np.array([0, 0, 1, 0, -1, 1, 1, -1, -1], dtype=float)
WGT = np.array([4 / 9] + [1 / 9] * 4 + [1 / 36] * 4)


@pytest.fixture(scope="module")
def sd():
    import torch
    assert torch.cuda.is_available(), "GPU tests need a HIP device"
    from paper_2007_07347_amd import sdugks
    return sdugks


def test_reciprocal_of_a_density_is_the_divisions(sd):
    """Equal bit by bit to 1 / x: densities spread over (0.5, 2) and over eight
    decades, and the numbers next to powers of two -- 1 / (1 - a 2^-53) for odd a
    lies a^2 2^-54 of an ulp from the middle of two numbers, where an error
    far below an ulp already rounds the wrong way."""
    rng = np.random.default_rng(3)
    a = np.arange(1, 1 << 16)
    near = np.concatenate([1.0 - a * 2.0 ** -53, 1.0 + a * 2.0 ** -52])
    x = np.concatenate([rng.uniform(0.5, 2.0, 1 << 20), 10.0 ** rng.uniform(-4, 4, 1 << 20),
                        *(near * 2.0 ** k for k in (-40, -3, 0, 1, 40))])
    y = sd.debug_reciprocal(x)
    bad = y != 1.0 / x
    assert not bad.any(), (bad.sum(), [float(v).hex() for v in x[bad][:4]])


@pytest.mark.parametrize("prec", ["FP64", "FP32DEV"])
@pytest.mark.parametrize("structured", [0, 1])
@pytest.mark.parametrize("n", [(8, 8), (32, 16), (256, 256), (768, 640)])
def test_a_foot_point_at_the_centre_reads_the_cell(sd, n, structured, prec):
    """Free transport (tau = 1e30) of a random f over a periodic box of squares of
    side h with dt = h / 2: the four velocities along the axes have their foot
    points x_f - e dt at the upwind cell's centre, so one step gives
    f - (f - f_upwind) / 2 whatever the slopes.  The reconstruction's offset from the
    centre is zero there and adds no rounding: the flux is the stored f exactly,
    and of the result's two operations in FP64 the second is rounded to the stored
    form, half an ulp.  What the equilibrium adds is below dt / tau = 1e-31.  fbar+
    carried back along e dt first and forth by the face's offset after misses
    that by up to an ulp of the slopes' contribution, several times f's."""
    nx, ny = n
    mesh, bcs = meshgen.periodic_box(nx, ny, lx=nx / 16.0, ly=ny / 16.0)
    h = 1 / 16.0
    s = sd.Solver(mesh, bcs, tau=1e30, dt=h / 2, precision=getattr(sd, prec), structured=structured)
    f, _, _ = meshgen.random_state(nx * ny, seed=5, amp=0.3)
    if prec == "FP32DEV":
        f = WGT + (f - WGT).astype(np.float32)          # f - w is stored exactly
        f = f.astype(np.float64)
    s.set_state(f, np.c_[f.sum(1), f @ EX, f @ EY])
    f0 = s.state()[0]
    s.step(1)
    f1 = s.state()[0]
    g = sd.geometry(mesh, bcs, tau=1e30, dt=h / 2)
    s.close()
    i, j = np.rint(g["cx"] / h - 0.5).astype(int), np.rint(g["cy"] / h - 0.5).astype(int)
    at = np.empty((nx, ny), int)
    at[i, j] = np.arange(nx * ny)
    d0 = f0 - WGT if prec == "FP32DEV" else f0
    d1 = f1 - WGT if prec == "FP32DEV" else f1
    for k, (ex, ey) in {1: (1, 0), 2: (0, 1), 3: (-1, 0), 4: (0, -1)}.items():
        up = at[(i - ex) % nx, (j - ey) % ny]
        want = d0[:, k] - 0.5 * (d0[:, k] - d0[up, k])
        # (f read back as w + the stored deviation, w in FP64: an FP64 ulp of f more)
        tol = 0.5 * np.spacing(np.abs(want).astype(np.float32)) if prec == "FP32DEV" else 0.5 * np.spacing(np.abs(want))
        tol = 1.000001 * tol.astype(float) + 4 * np.spacing(np.abs(f0[:, k]) + np.abs(f0[up, k]))
        assert np.all(np.abs(d1[:, k] - want) <= tol), (k, np.max(np.abs(d1[:, k] - want) / tol))
    # at rest: no flux
    assert np.all(np.abs(d1[:, 0] - d0[:, 0]) <= 2 * np.spacing(np.abs(f0[:, 0])))


def _start(n, seed, cx, cy):
    rng = np.random.default_rng(seed)
    return (1 + 0.02 * np.sin(3 * cx + seed) * np.cos(2 * cy), 0.05 * np.sin(4 * cy + seed) + 0.01 * rng.uniform(-1, 1, n),
            0.05 * np.cos(3 * cx) + 0.01 * rng.uniform(-1, 1, n))


def test_fp32_deviations_stay_near_fp64(sd):
    """Distance of f in FP32 deviations from f in FP64 after 1 and 200 steps of
    twenty periodic boxes (40 to 192 cells an edge, CFL 0.35 to 0.73): the geometric
    mean of its rms over the boxes.  The bounds are what one workgroup per tile with
    b feq weighted in FP64 and one offset to the foot point gave on the same boxes
    and states."""
    bound = {1: 2.921e-10, 200: 4.492e-10}
    err = {steps: [] for steps in bound}
    for k, n in enumerate(range(40, 200, 8)):
        mesh, bcs = meshgen.periodic_box(n, n)
        kw = dict(nu=1e-3, cfl=0.35 + 0.02 * k)
        g = sd.geometry(mesh, bcs, **kw)
        run = [sd.Solver(mesh, bcs, precision=p, **kw) for p in (sd.FP64, sd.FP32DEV)]
        done = 0
        for s in run:
            s.set_macros(*_start(s.n_cells, k, g["cx"], g["cy"]))
        for steps in bound:
            for s in run:
                s.step(steps - done)
            done = steps
            a, b = (s.state()[0] for s in run)
            err[steps].append(np.sqrt(((a - b) ** 2).mean()))
        for s in run:
            s.close()
    mean = {steps: float(np.exp(np.log(v).mean())) for steps, v in err.items()}
    print(mean, flush=True)
    assert all(mean[steps] <= bound[steps] for steps in bound), mean
