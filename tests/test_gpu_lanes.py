"""The kernels that walk neighbour rows give a particle 16, 4 or 1 lanes by
the size of the system; the sums are the same bits.  A box is replicated in
one batch until the launches pass each limit: every copy (same seed, same
particles, so the same motion and the same searches) must keep the bits the
box gets alone."""
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


def _box(kind):
    if kind == "tank":  # walls, free surface, spheres in contact, no noise
        p, parts, info = W.dam_break(tank=(22, 11, 18), column=(11, 11, 13), n_rigid=10, seed=4)
        return p, W.perturb(parts, p, jitter=0.1, kT=4e-2, seed=9, spin=True), info
    p, parts, info = W.shear_cell(15, phi=0.15, d=2.5, kBT=4e-3, shear_rate=8e-2, seed=5)
    return p, W.perturb(parts, p, jitter=0.1, kT=None, seed=9), info


def _state(g, n, copies, stress):
    out = {f: g.read_field(f).reshape(copies, n, -1)
           for f in ("POS", "VEL", "ANGVEL", "DENS", "PRES_SMOOTH", "F_SDPD", "N_SDPD", "F_CD")}
    rows, cols = g.read_neighbors()
    out["rowlen"] = np.diff(rows).reshape(copies, n)
    if stress:
        out["stress"] = g.box_stress()[1].reshape(copies, 1)
    return out, cols


@pytest.mark.parametrize("skin", [0.0, 0.2])
@pytest.mark.parametrize("kind", ["tank", "shear"])
def test_bits_do_not_depend_on_the_lanes_per_particle(S, kind, skin):
    cell = _box(kind)
    p, n = dict(cell[0], cell_factor=0.55, skin=skin), cell[1]["id"].shape[0]
    assert n <= 1 << 14  # 16 lanes alone
    ref = None
    for total in (n, 60_000, 150_000, 300_000, 450_000, 900_000):
        copies = max(1, -(-total // n))
        parts, boxes, box_of = W.stack_cells([cell] * copies)
        print(f"[case] {kind} x {copies}, n={copies * n}, skin {skin}", flush=True)
        g = S.System(p, parts, boxes=boxes, box_of=box_of)
        g.set_stress(kind == "shear")
        assert g.step(12) == 0
        got, cols = _state(g, n, copies, kind == "shear")
        if ref is None:
            ref, ref_cols = got, cols
            if skin:
                assert g.info()[14] > 0  # some lists came from the candidates
        for f, v in got.items():
            for b in (0, copies // 2, copies - 1):
                assert np.array_equal(v[b], ref[f][0]), (f, b)
        assert np.array_equal(cols[:ref_cols.size], ref_cols)
        assert np.array_equal(cols[-ref_cols.size:] - (copies - 1) * n, ref_cols)
        g.close()


def _narrow(kind, nx):
    """A jittered box nx cells of 1.05 h across in x; walls in z for "walls"."""
    h, L = 1.5, 1.5 * 1.05 * nx
    p, parts, info = W.random_box(int(0.8 * L * 9.0 * 9.0), (L, 9.0, 9.0),
                                  (1, 1, 0 if kind == "walls" else 1), h=h, seed=nx)
    # late enough for the images across the sheared faces to be displaced
    p = dict(p, kBT=4e-3, shear_rate=6e-2 if kind == "shear" else 0.0, itr_start=12345)
    if kind == "walls":  # outer walls in every cell, binned behind the fluid
        parts["type"][::9] = W.OUTER_WALL
    return p, parts, info


@pytest.mark.parametrize("skin", [0.0, 0.1])
@pytest.mark.parametrize("kind,nx,cf", [("plain", 3, 1.0), ("plain", 4, 1.0), ("walls", 3, 1.0),
                                        ("shear", 3, 1.0), ("shear", 4, 1.0), ("shear", 5, 1.0),
                                        ("shear", 6, 1.0), ("plain", 3, 0.55), ("shear", 3, 0.55)])
def test_bits_of_narrow_boxes(S, kind, nx, cf, skin):
    """Rows of the search that take the x axis whole start at cell 0 in every
    kernel: three to six cells across, of h or more (reach 1) and less."""
    cell = _narrow(kind, nx)
    p, n = dict(cell[0], cell_factor=cf, skin=skin), cell[1]["id"].shape[0]
    assert n <= 1 << 14  # 16 lanes alone
    ref = None
    for total in (n, 60_000, 870_000 if kind == "shear" else 620_000):  # 16 lanes, 4, 1
        copies = max(1, -(-total // n))
        parts, boxes, box_of = W.stack_cells([cell] * copies)
        print(f"[case] {kind}, {nx} cells, cell factor {cf}, skin {skin}, x {copies}", flush=True)
        g = S.System(p, parts, boxes=boxes, box_of=box_of)
        assert g.compute_forces() == 0
        got, _ = _state(g, n, copies, False)
        if ref is None:
            ref = got
        for f, v in got.items():
            for b in (0, copies // 2, copies - 1):
                assert np.array_equal(v[b], ref[f][0]), (f, b)
        g.close()


@pytest.mark.parametrize("skin", [0.0, 0.2])
def test_bits_do_not_depend_on_the_waves_per_sphere(S, skin):
    """One large sphere per box, whose coupling takes some eighteen rounds of
    a wave: a workgroup per sphere alone, a wave in a batch of more than 1024."""
    cell = W.shear_cell(13, phi=0.1, d=7.0, kBT=4e-3, shear_rate=5e-2, seed=6)
    n = cell[1]["id"].shape[0]
    assert int((cell[1]["type"] == W.RIGID).sum()) == 1
    p = dict(cell[0], cell_factor=0.55, skin=skin)
    ref = None
    for copies in (1, 1030):
        parts, boxes, box_of = W.stack_cells([cell] * copies)
        print(f"[case] sphere of radius 3.5 x {copies}, skin {skin}", flush=True)
        g = S.System(p, parts, boxes=boxes, box_of=box_of)
        g.set_stress(True)
        assert g.step(8) == 0
        got = {f: g.read_field(f).reshape(copies, n, -1)
               for f in ("VEL", "F_DG", "F_PG", "F_RXN", "EPS")}
        got["stress"] = g.box_stress()[1].reshape(copies, 1)
        ref = ref or got
        for f, v in got.items():
            for b in (0, copies // 2, copies - 1):
                assert np.array_equal(v[b], ref[f][0]), (f, b)
        g.close()


def _fluid(kind):
    if kind == "shear":
        p, parts, info = W.shear_cell(15, phi=0.0, kBT=4e-3, shear_rate=8e-2, seed=5)
    elif kind == "thermal":  # driven both ways, half of the box each
        p, parts, info = W.reverse_poiseuille((14, 15, 16), kBT=4e-2, g=1e-2, seed=3)
    else:  # a column under gravity that strikes its walls, no noise
        p, parts, info = W.dam_break(tank=(12, 11, 14), column=(12, 11, 9), n_rigid=0)
        p = dict(p, noslip=int(kind == "noslip"), g=[2e-2, 1e-2, -5e-2])
    kT = 2.0 if kind in ("slip", "noslip") else 4e-2  # fast enough to cross a wall
    return p, W.perturb(parts, p, jitter=0.1, kT=kT, seed=9, spin=True), info


@pytest.mark.parametrize("copies", [1, 12, 60])  # 16 lanes, 4, and (thermal) one
@pytest.mark.parametrize("skin", [0.0, 0.2])
@pytest.mark.parametrize("kind", ["shear", "thermal", "slip", "noslip"])
def test_the_update_in_the_pair_kernel_keeps_the_bits(S, kind, skin, copies):
    """Without spheres the pair kernel of a step's first pass updates its
    particles; while the virial is accumulated, a kernel of its own does."""
    cell = _fluid(kind)
    p = dict(cell[0], cell_factor=0.55, skin=skin)
    got = []
    for stress in (False, True):
        parts, boxes, box_of = W.stack_cells([cell] * copies)
        print(f"[case] {kind} x {copies}, skin {skin}, stress {stress}", flush=True)
        g = S.System(p, parts, boxes=boxes, box_of=box_of)
        g.set_stress(stress)
        assert g.step(25) == 0
        got.append({f: g.read_field(f)
                    for f in ("POS", "VEL", "ANGVEL", "DENS", "F_SDPD", "N_SDPD")})
        got[-1]["searches"] = np.asarray(g.info()[14])
        g.close()
    for f, v in got[0].items():
        assert np.array_equal(v, got[1][f]), f


@pytest.mark.parametrize("n", [1, 63, 64, 65, 130, 700, 2000])
@pytest.mark.parametrize("order", ["as drawn", "by x", "lane 1 in cell 0"])
def test_binning_by_runs(S, n, order):
    """Runs of equal cells within a wave, at its edges, and none at all: every
    particle is found once, with the neighbours of the exact test."""
    L, h = 8.0, 1.5
    p, parts, _ = W.random_box(n, (L, L, L), (1, 1, 1), h=h, seed=n)
    if order == "by x":
        parts["pos"] = parts["pos"][np.lexsort(np.floor(parts["pos"] / 2.0).T[::-1])]
    elif order == "lane 1 in cell 0":
        parts["pos"][1::64] *= 1e-2
    x = parts["pos"]
    e = x[:, None] - x[None]
    e -= L * np.round(e / L)
    near = (e * e).sum(2) < h * h
    np.fill_diagonal(near, False)
    for cf in (0.55, 1.0):
        print(f"[case] n={n}, {order}, cell factor {cf}", flush=True)
        g = S.System(dict(p, cell_factor=cf, max_neighbors=160), parts)
        g.compute_forces()
        assert np.array_equal(g.read_field("POS").reshape(n, 3), x)
        rows, cols = g.read_neighbors()
        got = np.zeros_like(near)
        got[np.repeat(np.arange(n), np.diff(rows)), cols] = True
        assert np.array_equal(got, near) and len(cols) == near.sum()
        g.close()
