"""Sixteen and thirty-two lanes per atom in the LJ kernel, and lane counts whose items take
several passes (more than 8,192 atoms): energies, forces and virials against the oracle."""
import numpy as np
import pytest

from gpu_cases import TOL_E_PER_ATOM, TOL_F, TOL_V_PER_ATOM, oracle_params_like

pytestmark = pytest.mark.gpu


@pytest.mark.parametrize("cells,lanes,fp64", [(2, 32, False), (4, 16, False), (4, 32, True), (6, 16, True), (6, 32, False),
                                              (13, 8, False), (13, 16, False)])
def test_lanes_and_passes(cells, lanes, fp64, monkeypatch):
    import oracle
    import torch
    import workloads as W
    from paper_2510_16721_amd import cfneb
    if not torch.cuda.is_available():
        pytest.skip("no HIP device")
    w = W.fcc_vacancy_hop(cells, cells, cells, 1.5496)
    monkeypatch.setenv("CFNEB_LJ_LANES", str(lanes))
    g = cfneb.Band(cfneb.default_params(cfneb.CFNEB_LJ, force_fp64=int(fp64), n_images=3, max_images=3), w["pos_init"],
                   w["cell_init"], w["pos_final"], w["cell_final"])
    monkeypatch.delenv("CFNEB_LJ_LANES")
    g.step(2)
    assert g.step(1, 1e30)[2]  # evaluate, no move
    img = g.image(1)
    E, _, F, V = oracle.evaluate(oracle_params_like("lj"), img["R"], img["h"])
    scale = 1e-6 if fp64 else 1.0
    assert abs(img["E"] - E) / g.n <= TOL_E_PER_ATOM * scale
    assert np.abs(img["F"] - F).max() <= TOL_F * scale
    assert np.abs(img["V"] - V).max() / g.n <= TOL_V_PER_ATOM * scale
    g.close()
