"""Timing a kernel changes no result, whichever launches of a step it separates."""
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


@pytest.mark.parametrize("skin", [0.0, 0.2])
@pytest.mark.parametrize("kT", [0.0, 1e-3])
def test_bits_do_not_depend_on_the_timed_kernel(S, kT, skin):
    p, parts, _ = W.reverse_poiseuille((14, 15, 16), kBT=kT, seed=3)
    parts = W.perturb(parts, p, jitter=0.1, kT=4e-2, seed=9, spin=True)
    ref = None
    for kernel, every, timed in (("none", 1, 0), ("fluid_forces", 1, 14), ("fluid_forces", 3, 5),
                                 ("integrate", 1, 14), ("smooth", 1, None)):
        print(f"[case] kT {kT}, skin {skin}, {kernel}, one in {every}", flush=True)
        g = S.System(dict(p, skin=skin), parts)
        g.set_profiling(kernel, every=every)
        assert g.step(7) == 0
        if timed is not None:
            assert g.kernel_time()[1] == timed
        got = {f: g.read_field(f) for f in ("POS", "VEL", "ANGVEL", "DENS", "F_SDPD", "N_SDPD")}
        g.close()
        ref = ref or got
        for f, v in got.items():
            assert np.array_equal(v, ref[f]), f
