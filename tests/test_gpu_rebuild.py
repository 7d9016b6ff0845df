"""Lists rebuilt inside a step call, where the bins change hands (a block per image for all of
it, a block per image for the bins, four launches): the moving images have gone further than the
skin allows, so the list of the creation cannot be the one in use, and the neighbour sets are
the oracle's, bit for bit."""
import numpy as np
import pytest

from test_gpu_bins import _check, _positions

pytestmark = pytest.mark.gpu


@pytest.mark.parametrize("n", [300, 4096, 4097, 36864, 36865])
def test_rebuilt_in_a_step(n):
    import torch
    from paper_2510_16721_amd import cfneb
    if not torch.cuda.is_available():
        pytest.skip("no HIP device")
    pos, h = _positions(n, 0.6, np.random.default_rng(n))
    skin = 0.004  # (small: these structures relax by a hundredth in a few hundred steps)
    p = cfneb.default_params(cfneb.CFNEB_LJ, n_images=4, max_images=4, lj_sigma=0.4, lj_rc=1.3, nbr_skin=skin, nbr_cap=200)
    band = cfneb.Band(p, pos, h, pos + 0.01, h @ (np.eye(3) * 1.003))
    before = [band.image(k) for k in (1, 2)]

    def gone():  # the least over the images of their largest move beyond the cell's strain
        now = [band.image(k) for k in (1, 2)]
        return min(np.linalg.norm(b["R"] - a["R"] @ np.linalg.solve(a["h"], b["h"]), axis=1).max()
                   for a, b in zip(before, now))

    for _ in range(20):
        band.step(12, 0.0)
        if 2.0 * gone() > skin:
            break
    assert 2.0 * gone() > skin
    _check(band, 1, 1.3)
    _check(band, 2, 1.3)
    band.close()


@pytest.mark.parametrize("fp64", [False, True])
def test_crowded_and_not_in_turn(fp64):
    # moving carbon atoms that get more than four bonds, lose them and get them again, in bands
    # that keep their state: what a band made with the last coordinates gives, and the oracle,
    # the atoms far from the crowded ones against their own scale
    import oracle
    import torch
    from gpu_cases import TOL_F, oracle_params_like
    from paper_2510_16721_amd import cfneb
    from test_gpu_crowded_items import _crowd, _diamond, _far
    if not torch.cuda.is_available():
        pytest.skip("no HIP device")
    pos, h = _diamond()
    n = len(pos)
    rng = np.random.default_rng(8)
    centres = rng.choice(n, 30, replace=False)
    a, b = _crowd(pos, h, centres[:20]), _crowd(pos, h, centres[10:])
    p = cfneb.default_params(cfneb.CFNEB_TERSOFF_C, force_fp64=int(fp64), n_images=3, max_images=3, nbr_cap=32)

    def run(states):
        g = cfneb.Band(p, pos, h, pos + 0.01, h)
        st = g.get_state()
        for x in states:
            st["X"][1, :n] = x
            g.set_state(st["X"], st["v"], st["dt"], st["alpha"], st["n_pos"], st["fresh"], st["step"], st["ci"])
            assert g.step(1, 1e30)[2]  # an evaluation without a move
            g.neighbours(1)  # (packs every image's counts)
        img = g.image(1)
        g.close()
        return img

    for last, moved in ((pos, a[1]), b):
        img, fresh = run([a[0], b[0], pos, a[0], last]), run([last])
        assert img["E"] == fresh["E"]
        np.testing.assert_array_equal(img["V"], fresh["V"])
        np.testing.assert_array_equal(img["F"], fresh["F"])
        E, _, F, V = oracle.evaluate(oracle_params_like("ts"), img["R"], img["h"])
        # as the crowded shells' test: rounding of some n^2 terms in FP64; 2^-24 on the bond lengths,
        # amplified by the exponents, in FP32, against the largest value
        tol = 1e-11 if fp64 else 2e-5
        assert abs(img["E"] - E) <= tol * abs(E)
        assert np.abs(img["F"] - F).max() <= tol * max(1.0, np.abs(F).max())
        assert np.abs(img["V"] - V).max() <= tol * max(float(n), np.abs(V).max())
        far = _far(pos, h, moved)
        assert far.any() and np.abs(img["F"] - F)[far].max() <= TOL_F * (1e-6 if fp64 else 1.0)
