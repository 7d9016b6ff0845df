"""Endpoints that differ by a translation alone: the springs' squared lengths are zero up to the
rounding of sums of either sign, and the band's evaluation is that of its structure."""
import numpy as np
import pytest

from gpu_cases import TOL_E_PER_ATOM, oracle_params_like

pytestmark = pytest.mark.gpu


@pytest.mark.parametrize("fp64", [False, True])
@pytest.mark.parametrize("kind,cells,images", [("lj", 3, 5), ("lj", 6, 12), ("ts", 2, 12), ("ts", 4, 7), ("ts", 8, 12)])
def test_translated_endpoints(kind, cells, images, fp64):
    import oracle
    import torch
    import workloads as W
    from paper_2510_16721_amd import cfneb
    if not torch.cuda.is_available():
        pytest.skip("no HIP device")
    w = W.fcc_vacancy_hop(cells, cells, cells) if kind == "lj" else W.diamond_vacancy_hop(cells, cells, cells)
    pos, h = w["pos_init"], w["cell_init"]
    p = cfneb.default_params(cfneb.CFNEB_LJ if kind == "lj" else cfneb.CFNEB_TERSOFF_C, force_fp64=int(fp64),
                             n_images=images, max_images=images)
    g = cfneb.Band(p, pos, h, pos + 0.01, h)
    assert g.step(1, 1e30)[2]  # an evaluation without a move
    E = oracle.evaluate(oracle_params_like(kind), pos, h)[0]
    tol = TOL_E_PER_ATOM * (1e-6 if fp64 else 1.0)  # (about 7 eV an atom: 1e-12 is some thousand roundings)
    assert np.abs(g.energies()["H"] - E).max() / len(pos) <= tol
    g.close()
