"""Contact partner lists and the reaction of dense suspensions against the
FP64 oracle.  A list row holds up to 63 partners; spheres with more search
the rigid grid in every pass, and fluid particles coupled to more than 16
spheres search it for their reaction.  With candidate reuse the lists and
the grid stay those of the last search while the spheres move on."""
import math

import numpy as np
import pytest

from _parity import VECTOR_FIELDS, assert_force_field, assert_same_neighbors, assert_scalar_fields
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


def _suspension(m, shear, seed):
    """A 9^3 fluid lattice and m^3 spheres of radius 1/4, jittered so that a
    few overlap; m = 10, 11 and 12 put about 46, 61 and 79 partners within
    R_s + R_k + h."""
    rng = np.random.default_rng(seed)
    p, fluid, _ = W.shear_cell(9, phi=0.0, d=0.0, kBT=1e-3, shear_rate=shear, dt=5e-4, seed=seed)
    R, a = 0.25, 9.0 / m
    g = np.stack(np.meshgrid(*[np.arange(m)] * 3, indexing="ij"), -1).reshape(-1, 3)
    c = (g + 0.5) * a + rng.uniform(-1.0, 1.0, (m ** 3, 3)) * (0.5 * (a - 2 * R) + 0.01)
    c = np.mod(c, 9.0)
    n, ms = m ** 3, 2.5 * math.pi * (2 * R) ** 3 / 6.0
    vel = rng.normal(size=(n, 3)) * 1.5
    vel[:, 0] += shear * (c[:, 2] - 4.5)
    new = dict(type=np.full(n, W.RIGID, np.uint8), pos=c, vel=vel,
               angvel=rng.normal(size=(n, 3)), mass=np.full(n, ms),
               inertia=np.full(n, 0.4 * ms * R * R), radius=np.full(n, R))
    parts = {k: np.concatenate([fluid[k], v]) for k, v in new.items()}
    parts["id"] = np.arange(parts["type"].size, dtype=np.int64)
    return dict(p, max_contacts=32), parts


@pytest.mark.parametrize("skin", [0.0, 0.2])
@pytest.mark.parametrize("m,shear", [(10, 0.0), (11, 0.0), (12, 0.0), (11, 0.2), (12, 0.2)])
def test_dense_small_spheres_match_the_oracle(S, oracle_lib, m, shear, skin):
    p, parts = _suspension(m, shear, seed=m)
    print(f"[case] {m}^3 spheres of radius 1/4, shear {shear}, skin {skin}", flush=True)
    g = S.System(dict(p, skin=skin), parts)
    assert g.step(120) == 0
    info = g.info()
    print(f"  {info[13]} searches, {info[14]} lists from candidates", flush=True)
    if skin:
        assert info[13] >= 2 and info[14] >= 30
    state = {k: np.array(v, copy=True) for k, v in parts.items()}
    state["pos"], state["vel"], state["angvel"] = (g.read_field(f) for f in
                                                   ("POS", "VEL", "ANGVEL"))
    o = oracle_lib.Oracle(dict(p, itr_start=g.current_step), state)
    pairs, dts = g.read_contacts()
    assert len(pairs) > 0
    o.load_contacts(pairs, dts)
    assert g.compute_forces(check=False) == o.compute_forces(check=False) == 0
    assert_same_neighbors(g, o)
    assert_scalar_fields(g, o, p)
    for f in VECTOR_FIELDS:
        assert_force_field(g, o, f)
    # the next committed contact table holds the same pairs
    assert g.step(1) == o.step(1) == 0
    pg, dg = g.read_contacts()
    po, do = o.read_contacts()
    assert np.array_equal(pg, po)
    assert np.allclose(dg, do, rtol=0, atol=1e-7)
