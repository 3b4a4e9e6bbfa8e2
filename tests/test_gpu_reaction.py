"""The reaction of dense suspensions takes several lanes per fluid particle, a
rule over the whole batch: a dense box must keep its bits when dilute boxes of
the same batch move the launch to the one-lane form."""
import math

import numpy as np
import pytest

from paper_2002_03120_amd import workloads as W

pytestmark = pytest.mark.gpu


@pytest.fixture(scope="module")
def S():
    import torch
    if not torch.cuda.is_available():
        pytest.skip("no GPU")
    from paper_2002_03120_amd import sdpdem
    sdpdem.lib()
    return sdpdem


def _dense(L, m, shear):
    """An L^3 fluid lattice and m^3 jittered spheres of radius 1/4: some fifty
    spheres couple to a fluid particle, three times what its slots hold."""
    rng = np.random.default_rng(m)
    p, fluid, info = W.shear_cell(L, phi=0.0, d=0.0, kBT=1e-3, shear_rate=shear, dt=5e-4, seed=m)
    R, a = 0.25, L / m
    g = np.stack(np.meshgrid(*[np.arange(m)] * 3, indexing="ij"), -1).reshape(-1, 3)
    c = np.mod((g + 0.5) * a + rng.uniform(-1.0, 1.0, (m ** 3, 3)) * (0.5 * (a - 2 * R) + 0.01), L)
    n, ms = m ** 3, 2.5 * math.pi * (2 * R) ** 3 / 6.0
    vel = rng.normal(size=(n, 3)) * 1.5
    vel[:, 0] += shear * (c[:, 2] - 0.5 * L)
    new = dict(type=np.full(n, W.RIGID, np.uint8), pos=c, vel=vel,
               angvel=rng.normal(size=(n, 3)), mass=np.full(n, ms),
               inertia=np.full(n, 0.4 * ms * R * R), radius=np.full(n, R))
    parts = {k: np.concatenate([fluid[k], v]) for k, v in new.items()}
    parts["id"] = np.arange(parts["type"].size, dtype=np.int64)
    # late enough for the images across the sheared faces to be displaced
    return dict(p, max_contacts=32, itr_start=12345), parts, info


@pytest.mark.parametrize("skin", [0.0, 0.2])
@pytest.mark.parametrize("shear", [0.0, 0.2])
@pytest.mark.parametrize("L,m", [(6, 8), (9, 12)])  # rigid grids of 3 and 5 cells
def test_a_dense_box_keeps_its_bits_among_dilute_ones(S, L, m, shear, skin):
    cell = _dense(L, m, shear)
    water = W.shear_cell(12, phi=0.0, d=0.0, kBT=1e-3, shear_rate=shear, dt=5e-4, seed=1)
    n, p = cell[1]["id"].size, dict(cell[0], skin=skin)
    assert 22.4 * m ** 3 > 10 * L ** 3  # coupled spheres per fluid particle
    got = []
    for extra in (0, 4):
        assert extra == 0 or 22.4 * m ** 3 < 10 * (L ** 3 + extra * 12 ** 3)
        parts, boxes, box_of = W.stack_cells([cell] + [water] * extra)
        print(f"[case] {m}^3 spheres in {L}^3, shear {shear}, skin {skin}, {extra} boxes of fluid",
              flush=True)
        g = S.System(p, parts, boxes=boxes, box_of=box_of)
        assert g.step(6) == 0
        got.append({f: g.read_field(f).reshape(g.n, -1)[:n] for f in ("F_RXN", "VEL", "POS")})
        g.close()
    for f, v in got[0].items():
        assert np.array_equal(v, got[1][f]), f


@pytest.mark.parametrize("extra", [0, 4])  # several lanes per particle, one
def test_a_sphere_out_of_reach_adds_nothing(S, extra):
    """A sphere so fast that its drag overflows: the reaction of the fluid
    beyond its support stays what it is without that sphere's drag."""
    L, m = 9, 12
    p, parts, _ = _dense(L, m, 0.0)
    n, s = parts["id"].size, int(np.flatnonzero(parts["type"] == W.RIGID)[0])
    parts["vel"][s] = 1e200
    e = parts["pos"] - parts["pos"][s]
    e -= L * np.round(e / L)
    far = (parts["type"] == W.FLUID) & ((e * e).sum(1) > (0.25 + p["h"]) ** 2)
    assert far.sum() > 100
    water = W.shear_cell(12, phi=0.0, d=0.0, kBT=1e-3, shear_rate=0.0, dt=5e-4, seed=1)
    parts, boxes, box_of = W.stack_cells([(p, parts, None)] + [water] * extra)
    print(f"[case] {m}^3 spheres in {L}^3, one at 1e200, {extra} boxes of fluid", flush=True)
    g = S.System(p, parts, boxes=boxes, box_of=box_of)
    g.compute_forces(check=False)
    f = g.read_field("F_RXN")[:n]
    g.close()
    assert np.isfinite(f[far]).all()
    assert not np.isfinite(f[(parts["type"][:n] == W.FLUID) & ~far]).all()
