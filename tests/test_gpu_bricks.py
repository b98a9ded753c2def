"""The push sweep by bricks, at the velocity counts and widths that the rule
gives them: against the oracle, and bit for bit where the sums have an order."""
import numpy as np
import pytest

import oracle
from paper_2412_06546_amd import cases

pytestmark = pytest.mark.gpu


def _gpu():
    import torch
    assert torch.cuda.is_available(), "these tests need the GPU"
    from paper_2412_06546_amd import ugks
    return ugks


def _cut(case, n, scatter=False):
    """The case with the n points nearest the origin of a grid, spread by a
    seeded jitter when no coordinates are to be shared."""
    dim = int(case["mesh"]["dim"])
    per_axis = max(2, int(np.ceil((1.02 * n) ** (1.0 / dim))) + 1)
    vg = cases.tensor_vgrid(per_axis, 4.0, dim)
    keep = np.sort(np.argsort((vg["u"] ** 2).sum(1), kind="stable")[:n])
    u, w = vg["u"][keep], vg["w"][keep]
    if scatter:
        u = u + np.random.default_rng(3).uniform(-0.03, 0.03, u.shape)
    return dict(case, vgrid=dict(dim=dim, u=np.ascontiguousarray(u), w=np.ascontiguousarray(w)))


def _match(c, sweep, steps=2):
    """FP64 rounding over the steps: the parity tests' 1e-12, W over its largest
    value (momentum over at least the density), q over at least
    p c = rho T / 2 sqrt(5 T / 6)."""
    s, o = _gpu().Solver(c, sweep=sweep), oracle.Oracle(c)
    s.step(steps)
    o.step(steps)
    Wg, qg = s.macros()
    Wo, qo = o.macros()
    T = (4.0 / 3.0) * (Wo[:, -1] - 0.5 * (Wo[:, 1:-1] ** 2).sum(1) / Wo[:, 0]) / Wo[:, 0]
    scale = np.abs(Wo).max(axis=0)
    scale[1:-1] = np.maximum(scale[1:-1], Wo[:, 0].max())
    pc = (0.5 * Wo[:, 0] * T * np.sqrt(5.0 * T / 6.0)).max()
    assert (np.abs(Wg - Wo).max(axis=0) / scale).max() <= 1e-12
    assert np.abs(qg - qo).max() / max(np.abs(qo).max(), pc) <= 1e-12


@pytest.mark.parametrize("sweep,n,nv,scatter", [
    ("push_unordered", 21, 450, False),   # 9,261 cells, the last brick holds one; 512 threads once
    ("push_unordered", 21, 512, False),
    ("push_unordered", 21, 701, False),   # 768 threads once
    ("push_unordered", 21, 1000, False),  # 512 threads twice
    ("push_unordered", 21, 1331, False),  # 768 threads twice
    ("push_unordered", 21, 861, True),    # scattered: 512 threads
    ("push", 33, 1337, False),            # 35,937 cells in colours, the small classes split
])
def test_bricks_match_the_oracle_3d(sweep, n, nv, scatter):
    print(f"case channel {n}^3, {nv} velocities, {sweep}", flush=True)
    _match(_cut(cases.case_channel_3d(n=n, kind="hex", nv=4), nv, scatter), sweep)


@pytest.mark.parametrize("sweep,nx,ny,nv,scatter", [
    ("push_unordered", 64, 65, 351, False),
    ("push_unordered", 64, 65, 784, False),
    ("push_unordered", 64, 65, 701, True),
    ("push", 128, 129, 350, False),
    ("push", 128, 129, 600, False),
    ("push", 128, 129, 701, True),
])
def test_bricks_match_the_oracle_2d(sweep, nx, ny, nv, scatter):
    print(f"case wave {2 * nx * ny}, {nv} velocities, {sweep}", flush=True)
    _match(_cut(cases.case_periodic_wave(nx=nx, ny=ny, nv=4), nv, scatter), sweep)


def test_tables_up_to_the_limit():
    """A set of 1,337 points over 249 coordinate values: tables and sums take
    80,352 of the 81,920 bytes of LDS that a brick's workgroup may."""
    c = cases.case_channel_3d(n=21, kind="hex", nv=4)
    rng = np.random.default_rng(11)
    axis = np.linspace(-4.0, 4.0, 83)
    at = np.concatenate([np.repeat(np.arange(83)[:, None], 3, axis=1), rng.integers(0, 83, (1254, 3))])
    vg = dict(dim=3, u=np.ascontiguousarray(axis[at]), w=np.full(1337, 512.0 / 1337))
    print("case channel 21^3, 1,337 points over 249 values, push_unordered", flush=True)
    _match(dict(c, vgrid=vg), "push_unordered", steps=1)


@pytest.mark.parametrize("mesh,nv,scatter", [("body", 1337, False), ("prism", 1600, False), ("triangles", 701, True)])
def test_coloured_bricks_are_deterministic(mesh, nv, scatter):
    """Two runs agree bit for bit on meshes with cells that fit in no whole
    brick, which follow the bricks in their classes, with several iterations a
    workgroup and with split classes."""
    ugks = _gpu()
    if mesh == "body":  # 34,083 cells, prisms and hexahedra
        c = cases.case_lifting_body(n=16, n_r=21, n_prism_columns=87, ma=0.5, t_wall=1.0)
    elif mesh == "prism":  # 35,152 cells (1,600 velocities go by cells)
        c = cases.case_channel_3d(n=26, kind="prism", nv=4)
    else:
        c = cases.case_periodic_wave(nx=128, ny=129, nv=4)
    c = _cut(c, nv, scatter)
    print(f"case {mesh}, {nv} velocities", flush=True)
    got = []
    for _ in range(2):
        s = ugks.Solver(c, sweep="push")
        s.step(3)
        got.append((*s.macros(), s.f()))
        s.close()
    for a, b in zip(*got):
        assert np.array_equal(a, b)
