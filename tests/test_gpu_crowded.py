"""Carbon atoms with more than four bonds: five to eight (eight lanes each), nine to sixty-four
(a wave) and more (a thread), alone in a wave and crowding it, against the oracle."""
import numpy as np
import pytest

from gpu_cases import oracle_params_like

pytestmark = pytest.mark.gpu


def _cluster(n, radius, seed, sep):
    rng = np.random.default_rng(seed)
    out = [np.zeros(3)]
    while len(out) < n:
        x = rng.uniform(-radius, radius, 3)
        if np.linalg.norm(x) < radius and min(np.linalg.norm(x - y) for y in out) > sep:
            out.append(x)
    return np.array(out)


@pytest.mark.parametrize("fp64", [False, True])
@pytest.mark.parametrize("n,radius,sep", [(6, 1.4, 0.9), (8, 1.5, 0.9), (9, 1.5, 0.9), (10, 1.5, 0.85), (40, 2.0, 0.5),
                                          (65, 1.04, 0.2), (66, 1.04, 0.2), (150, 1.6, 0.2)])
def test_many_bonds(n, radius, sep, fp64):
    import oracle
    import torch
    from paper_2510_16721_amd import cfneb
    if not torch.cuda.is_available():
        pytest.skip("no HIP device")
    h = np.eye(3) * 14.0
    # the cluster, chains of carbon with two bonds, and a second cluster elsewhere
    chain = np.array([[3.0 + 1.45 * q, 11.0, 1.0 + 2.6 * w] for w in range(4) for q in range(5)])
    pos = np.concatenate([chain, _cluster(n, radius, 5, sep) + 4.0, _cluster(7, 1.4, 6, 0.9) + np.array([10.0, 4.0, 11.0])])
    p = cfneb.default_params(cfneb.CFNEB_TERSOFF_C, force_fp64=int(fp64), n_images=3, max_images=3, nbr_cap=160)
    g = cfneb.Band(p, pos, h, pos + 0.01, h)
    img = g.image(0)
    E, _, F, V = oracle.evaluate(oracle_params_like("ts"), img["R"], img["h"])
    # FP64: rounding of some n^2 terms; FP32: 2^-24 on the bond lengths, amplified by the
    # exponents' l1 r < 8 and summed over an atom's bonds, against the largest force
    tol = 1e-11 if fp64 else 2e-5
    assert abs(img["E"] - E) <= tol * max(1.0, abs(E))
    assert np.abs(img["F"] - F).max() <= tol * max(1.0, np.abs(F).max())
    assert np.abs(img["V"] - V).max() <= tol * max(1.0, np.abs(V).max())
    g.close()
