"""Neighbour sets where the bins change hands: a block per image for all of it, a block per
image for the bins, four launches; a round of the block cut short; more bins than atoms; a
list rebuilt in the course of a relaxation.  The oracle's sets, bit for bit."""
import numpy as np
import pytest

from gpu_cases import sort_entries

pytestmark = pytest.mark.gpu


def _check(band, k, rc):
    import oracle
    img = band.image(k)
    cnt, ent = band.neighbours(k)
    ref = oracle.nlist(img["R"], img["h"], rc)
    assert [int(c) for c in cnt] == [len(r) for r in ref]
    for i in range(len(ref)):
        np.testing.assert_array_equal(sort_entries(ent[i]), ref[i])


def _positions(n, spacing, rng):
    """n atoms on a jittered grid in random order, in a slightly triclinic cell."""
    m = int(np.ceil(n ** (1.0 / 3.0)))
    h = np.diag([m * spacing] * 3) + np.array([[0, 0, 0], [0.11, 0, 0], [-0.07, 0.13, 0]]) * m * spacing
    g = np.stack(np.meshgrid(*[np.arange(m)] * 3, indexing="ij"), -1).reshape(-1, 3)
    g = g[rng.permutation(len(g))[:n]]
    jitter = 0.1 if spacing < 1.0 else 0.4  # the sparse ones: few neighbours, more bins than atoms
    return ((g + 0.5 + rng.uniform(-jitter, jitter, g.shape)) / m) @ h, h


@pytest.mark.parametrize("n,spacing", [(1023, 0.6), (4095, 0.6), (4096, 3.0), (4097, 0.6), (4097, 3.0), (5121, 0.6),
                                       (8193, 0.6), (36863, 0.6), (36864, 3.0), (36865, 0.6)])
def test_bins_give_the_exact_sets(n, spacing):
    import torch
    from paper_2510_16721_amd import cfneb
    if not torch.cuda.is_available():
        pytest.skip("no HIP device")
    rng = np.random.default_rng(n)
    pos, h = _positions(n, spacing, rng)
    p = cfneb.default_params(cfneb.CFNEB_LJ, n_images=3, max_images=3, lj_sigma=0.4, lj_rc=1.3, nbr_cap=200)
    band = cfneb.Band(p, pos, h, pos + 0.01, h @ (np.eye(3) * 1.003))
    for k in (0, 1):
        _check(band, k, 1.3)
    # moves of half a skin and more in total: the moving image rebuilds on the way
    if spacing < 1.0:
        band.step(12, 0.0)
        _check(band, 1, 1.3)
