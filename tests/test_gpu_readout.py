"""The readout of a band at its edges: fewer and more intervals than the block has waves, the
most images, a tile's rows cut short, more tiles than a wave has lanes."""
import numpy as np
import pytest

pytestmark = pytest.mark.gpu


@pytest.mark.parametrize("images,cells", [(3, 2), (17, 4), (18, 4), (64, 3), (19, 26)])
def test_path_coordinate_and_barrier(images, cells):
    import oracle
    import torch
    from paper_2510_16721_amd import cfneb
    if not torch.cuda.is_available():
        pytest.skip("no HIP device")
    rng = np.random.default_rng(images)
    g = np.stack(np.meshgrid(*[np.arange(cells)] * 3, indexing="ij"), -1).reshape(-1, 3)
    pos, h = (g + 0.25) * 1.1, np.eye(3) * 1.1 * cells
    p = cfneb.default_params(cfneb.CFNEB_LJ, n_images=images, max_images=images, lj_rc=1.05, nbr_cap=64)
    band = cfneb.Band(p, pos, h, pos + rng.normal(0, 0.02, pos.shape), h * 1.01)
    band.displace_interior(rng.normal(0, 0.02, (images - 2,) + pos.shape))
    e = band.energies()
    # sums of 3 (n + 3) squares in another order: far below 1e-12 of the path
    np.testing.assert_allclose(e["xi"], oracle.path_coord(band.get_state()["X"], band.n), rtol=0, atol=1e-12)
    assert len(e["H"]) == images and e["barrier"] == e["H"].max() - e["H"][0]
